// Device-side stages of Search by triplet for gfx950 (wave64).
//
// One event is processed by one workgroup of B lanes.  Every stage is a pure
// function of the event state at the stage start (the paper's barrier between
// seeding and following, Section 3) and every choice is a minimum over unique
// keys, so the parallel evaluation order never changes the result.
//
// Per-event state lives in the workspace, in regions indexed by the event's
// absolute hit offset hb (capacity N = hits of the event):
//   hs      16-byte sorted hits {x, y, z, phi16 | id << 16} by sorted position
//   owner   one bit per hit: set once a track has taken the hit (the method
//           only ever asks whether a hit is flagged; which track holds it is
//           settled by the claim keys).  Memory form: by hit id
//   claim   u64 per hit: minimum claim key of the current stage, for the
//           memory form (by id) and for the stages that the LDS form settles
//           exactly (by sorted position)
//   link    two u16 per hit (LDS form: by sorted position; memory form: by id):
//           the previous hit of the owning track, and the record of the
//           accepted track whose key is this id
//   rec     memory form: 32-byte forming-track records (one per seed; <= N)
//           and a 16-byte auxiliary record each (search result, seed fit,
//           filter outcome).  LDS form: 16-byte final records
//   lists   memory form: six u16 lists (active tracks x2, final tracks,
//           unflagged positions x2, unflagged ranks).  LDS form: the ids by
//           sorted position
// The LDS form keeps its forming tracks in registers, and the sorted hits,
// flags and claims of the modules around a step in LDS.
// Hit ids, keys and record indices are 16-bit (events hold <= 65,535 hits).
// Per-event bases are uniform; per-lane offsets are 32-bit.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sbt.h"

namespace sbt {

constexpr uint16_t kNone = 0xFFFFu;
constexpr unsigned long long kNoClaim = ~0ull;

// forming-track record
struct Rec {
    float xb, yb, zb;   // last hit
    float tx, ty;       // slope of the last two hits
    uint16_t key;       // id of the seed's middle hit (unique per event)
    uint16_t h0, h1, h2;
    uint16_t last;      // id of the last hit
    uint8_t len;        // hits
    uint8_t last_t;     // traversal index of the last hit
};
static_assert(sizeof(Rec) == 32, "record layout");

// per-record auxiliary data
struct RecAux {
    uint32_t best;      // memory instantiation: search result (best id | position << 16, or ~0)
    float bsc;          // its scatter
    float chi2;         // tracklet fit of the seed
    uint32_t flag;      // filter outcome
};
static_assert(sizeof(RecAux) == 16, "auxiliary record layout");

// sorted hit: coordinates and phi16 | id << 16
struct alignas(16) Hit16 {
    float x, y, z;
    uint32_t qid;
};

// per-event counters
struct EvInfo {
    int32_t nt, nh;     // accepted tracks and their hits
    int32_t out_h;      // first output hit position (batch scan)
    int32_t st;         // SBT_EV_* status
    int32_t nfin;       // final records (plain form)
    int32_t out_t;      // first output track position (batch scan)
    int32_t pos;        // 1: the LDS form tracked it (plain form)
    int32_t pad;
};

// record flags
constexpr uint32_t kFlagCandidate = 2;  // tracklet candidate
constexpr uint32_t kFlagAccepted = 4;

// memory lists (stride = workspace hit capacity)
constexpr int kListAct0 = 0, kListAct1 = 1, kListFin = 2, kListFreeL = 3, kListFreeM = 4, kListFRank = 5;
constexpr int kLists = 6;

// Workspace: one base pointer; every array sits at a fixed multiple of the
// hit capacity H (a multiple of 256) or, after the per-hit arrays, of the
// event capacity E.  Per hit: rec 32 B, hs 16, aux 16, claim 8, keys 4 (sort
// keys of events too large for the LDS sort), link 4, st_toff 4 (per-event
// track hit offsets), six u16 lists 12, st_hits 2 (per-event compacted hit
// ids).  Then the flag bitmaps (event e's starts at word (hb >> 5) + e), the
// per-event counters, the event order (largest first), the work counter (and
// beside it the count of events set aside) and the list of events set aside.
struct Work {
    char *base;
    uint32_t H, E;
};

constexpr uint32_t kOffRec = 0, kOffHs = 32, kOffAux = 48, kOffClaim = 64, kOffKeys = 72, kOffLink = 76,
                   kOffToff = 80, kOffLists = 84, kOffStHits = 96, kHitBytes = 98;

__host__ __device__ inline uint64_t ws_owner(uint32_t H) { return (uint64_t)H * kHitBytes; }
__host__ __device__ inline uint64_t ws_ev(uint32_t H, uint32_t E) { return ws_owner(H) + (((uint64_t)H / 32 + E + 2) * 4 + 255) / 256 * 256; }
__host__ __device__ inline uint64_t ws_order(uint32_t H, uint32_t E) { return ws_ev(H, E) + (uint64_t)E * 32; }
__host__ __device__ inline uint64_t ws_counter(uint32_t H, uint32_t E) { return ws_order(H, E) + (uint64_t)E * 4; }
// events a first pass set aside for a second one
__host__ __device__ inline uint64_t ws_defer(uint32_t H, uint32_t E) { return ws_counter(H, E) + 256; }
__host__ __device__ inline uint64_t ws_bytes(uint32_t H, uint32_t E) { return ws_defer(H, E) + ((uint64_t)E * 4 + 255) / 256 * 256; }

__host__ __device__ inline EvInfo *ws_evinfo(const Work &W) { return (EvInfo *)(W.base + ws_ev(W.H, W.E)); }
__host__ __device__ inline int32_t *ws_orderp(const Work &W) { return (int32_t *)(W.base + ws_order(W.H, W.E)); }
__host__ __device__ inline unsigned int *ws_counterp(const Work &W)
{
    return (unsigned int *)(W.base + ws_counter(W.H, W.E));
}
// the number of events set aside, beside the work counter
__host__ __device__ inline unsigned int *ws_defer_countp(const Work &W) { return ws_counterp(W) + 1; }
__host__ __device__ inline int32_t *ws_deferp(const Work &W) { return (int32_t *)(W.base + ws_defer(W.H, W.E)); }
__host__ __device__ inline Hit16 *ws_hs(const Work &W) { return (Hit16 *)(W.base + (uint64_t)W.H * kOffHs); }
__host__ __device__ inline int32_t *ws_toff(const Work &W) { return (int32_t *)(W.base + (uint64_t)W.H * kOffToff); }
__host__ __device__ inline uint16_t *ws_sthits(const Work &W)
{
    return (uint16_t *)(W.base + (uint64_t)W.H * kOffStHits);
}

struct HitsArgs {
    int32_t n_events;
    int32_t n_hits;
    const int32_t *eo;
    const int32_t *mo;
    const float *x, *y, *z;   // binary32 structure of arrays, or
    const uint2 *h16;         // binary16 x, y, z, unused per hit (null for binary32)
};

struct OutArgs {
    int32_t *eto;
    int32_t *tho;
    int32_t *th;
    int32_t *status;
};

// element i of an array with a uniform base, addressed with a 32-bit offset
template <class T>
__device__ __forceinline__ T &at(T *p, uint32_t i)
{
    return *reinterpret_cast<T *>(reinterpret_cast<char *>(p) + i * (uint32_t)sizeof(T));
}
template <class T>
__device__ __forceinline__ const T &at(const T *p, uint32_t i)
{
    return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(p) + i * (uint32_t)sizeof(T));
}

// ---------------------------------------------------------------- phi16
// Simplified atan2 on 16 bits (Section 3, "Sort by phi"): atan(r), r in
// [0,1], as r * P(r^2) with a degree-4 polynomial fitted in float64 and
// rounded to binary32 (max error 1.2e-5 rad), folded into the full circle and
// scaled by 32768/pi with round-to-nearest-even, so -pi and +pi meet at 0x8000.
__device__ __forceinline__ uint16_t phi16(float x, float y)
{
    const float c0 = 0x1.ffee7ap-1f;
    const float c1 = -0x1.523b6cp-2f;
    const float c2 = 0x1.70f766p-3f;
    const float c3 = -0x1.5ccd12p-4f;
    const float c4 = 0x1.55871cp-6f;
    const float half_pi = 0x1.921fb6p+0f;
    const float pi = 0x1.921fb6p+1f;
    const float scale = 0x1.45f306p+13f;   // 32768 / pi
    // |x| and |y| differ from the comparison form in the sign of a zero only,
    // which never reaches the result
    const float a = __builtin_fabsf(x), b = __builtin_fabsf(y);
    const float mn = a < b ? a : b;
    float mx = a < b ? b : a;
    mx = mx == 0.0f ? 1.0f : mx;   // (0, 0) has angle 0
    const float r = mn / mx;
    const float s = r * r;
    float p = c4;
    p = p * s + c3;
    p = p * s + c2;
    p = p * s + c1;
    p = p * s + c0;
    float at = r * p;
    at = b > a ? half_pi - at : at;
    at = x < 0.0f ? pi - at : at;
    at = y < 0.0f ? -at : at;
    const int q = (int)__builtin_rintf(at * scale);
    return (uint16_t)(q & 0xFFFF);
}

// ---------------------------------------------------------------- small helpers
// Workgroup barrier that orders LDS accesses only: stores to memory issued
// before it are not waited for.  Used where the next phase reads nothing the
// previous one wrote to memory.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A value every lane of the wave holds alike (read from LDS, for instance),
// moved to a scalar register.
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Lane index among the lanes that run one event.  An event of 64 lanes is
// one wave, and a workgroup may hold several of them, one event per wave;
// wider events have their workgroup to themselves.
template <int B>
__device__ __forceinline__ int tid()
{
    return B == 64 ? (int)(threadIdx.x & 63u) : (int)threadIdx.x;
}

// Barrier over the lanes of one event.  The lanes of a 64-lane event are one
// wave and run in lockstep, so only its memory operations have to complete
// (the fences); the workgroup's other waves run other events and are not
// waited for.
template <int B>
__device__ __forceinline__ void ev_sync()
{
    if (B == 64) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    } else {
        __syncthreads();
    }
}

// The same for phases that exchange LDS data only (see lds_barrier).
template <int B>
__device__ __forceinline__ void ev_lds_sync()
{
    if (B == 64) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    } else {
        lds_barrier();
    }
}

// The value, hidden from the optimiser at this point.  Stages re-read the
// scalar parameters and the workspace base through this at the start of
// every module step, so values derived from them are recomputed per step
// instead of being hoisted out of the event and step loops, where dozens of
// them would stay live in scalar registers (and spill) for the whole kernel.
// Where a kernel's control flow leaves the compiler holding the value in a
// vector register, the readfirstlane brings it back to a scalar one, as the
// asm operand needs; elsewhere it costs nothing.
template <class T>
__device__ __forceinline__ T opq(T v)
{
    static_assert(sizeof(T) == 4, "one scalar register");
    int x = uni(__builtin_bit_cast(int, v));
    asm volatile("" : "+s"(x));
    return __builtin_bit_cast(T, x);
}

// A workspace pointer hidden from the optimiser (see opq) that stays known
// as global memory, so its accesses remain global (not flat) instructions.
typedef __attribute__((address_space(1))) char gchar;
__device__ __forceinline__ char *opq_global(char *p)
{
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    uint64_t v = ((uint64_t)(uint32_t)uni((int)(uint32_t)(a >> 32)) << 32) | (uint32_t)uni((int)(uint32_t)a);
    asm volatile("" : "+s"(v));
    return (char *)(gchar *)v;
}

// scalar parameters of the stages
struct Prm {
    int M, rev, K, Ws, Wf, misses;
    float Ss, Sf, X;
};

__device__ __forceinline__ Prm fresh(const sbt_params &P)
{
    Prm p;
    p.M = opq(P.n_modules);
    p.rev = opq(P.reverse);
    p.K = opq(P.max_doublet_candidates);
    p.Ws = opq(P.phi_window_seeding);
    p.Wf = opq(P.phi_window_forwarding);
    p.misses = opq(P.max_consecutive_misses);
    p.Ss = __int_as_float(opq(__float_as_int(P.max_scatter_seeding)));
    p.Sf = __int_as_float(opq(__float_as_int(P.max_scatter_forwarding)));
    p.X = __int_as_float(opq(__float_as_int(P.max_tracklet_chi2)));
    return p;
}

// The parameter block of the running kernel (its first argument), by an
// address hidden from the optimiser: each use is a scalar load where it
// stands, instead of registers held (and spilled) through the whole kernel.
typedef __attribute__((address_space(4))) const sbt_params cparams;
__device__ __forceinline__ const sbt_params &kernel_params()
{
    uint64_t a = reinterpret_cast<uint64_t>(__builtin_amdgcn_kernarg_segment_ptr());
    asm volatile("" : "+s"(a));
    return *(const sbt_params *)reinterpret_cast<cparams *>(a);
}

__device__ __forceinline__ int kmod(const Prm &p, int t) { return p.rev ? p.M - 1 - t : t; }
__device__ __forceinline__ int kmod(const sbt_params &P, int t)
{
    return P.reverse ? P.n_modules - 1 - t : t;
}

// largest k in [0, M) with mo[k] <= i (requires mo[0] <= i < mo[M])
__device__ __forceinline__ int module_of(const int *mo, int M, int i)
{
    int lo = 0, hi = M;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (mo[mid] <= i) lo = mid; else hi = mid;
    }
    return lo;
}

// hit flags: one bit per event-local hit id
__device__ __forceinline__ bool is_free(const uint32_t *own, unsigned id)
{
    return ((at(own, id >> 5) >> (id & 31u)) & 1u) == 0u;
}

__device__ __forceinline__ void set_flag(uint32_t *own, unsigned id)
{
    atomicOr(&at(own, id >> 5), 1u << (id & 31u));
}

// Claim key of a stage: (255 - stage) in bits 48..55, the score's binary32
// bits in 16..47 (scores are >= +0, so the bits order like the values) and
// the track key in 0..15.  Within a stage the order is (score, key); a claim
// left from an earlier stage is larger than any claim of a later one, so the
// claim words never need clearing between stages.
__device__ __forceinline__ unsigned long long claim_key(float score, uint16_t key, int stage)
{
    return ((unsigned long long)(255 - stage) << 48) | ((unsigned long long)__float_as_uint(score) << 16) | key;
}
constexpr int kFilterStage = 64;

// number of set bits of m below this lane
__device__ __forceinline__ int lane_rank(unsigned long long m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Append under a predicate with one LDS atomic per wave; every lane of the
// wave must call it.  Returns the slot, or -1 where pred is false.
__device__ __forceinline__ int wave_append(bool pred, int *counter)
{
    const unsigned long long m = __ballot(pred);
    if (m == 0) return -1;
    int base = 0;
    if (lane_rank(__builtin_amdgcn_read_exec()) == 0) base = atomicAdd(counter, __popcll(m));
    base = __builtin_amdgcn_readfirstlane(base);
    return pred ? base + lane_rank(m) : -1;
}

// Two appends at once (their atomics overlap); every lane must call it.
__device__ __forceinline__ void wave_append2(bool p0, int *c0, bool p1, int *c1, int &r0, int &r1)
{
    const unsigned long long m0 = __ballot(p0), m1 = __ballot(p1);
    int b0 = 0, b1 = 0;
    if (lane_rank(__builtin_amdgcn_read_exec()) == 0) {
        if (m0) b0 = atomicAdd(c0, __popcll(m0));
        if (m1) b1 = atomicAdd(c1, __popcll(m1));
    }
    b0 = __builtin_amdgcn_readfirstlane(b0);
    b1 = __builtin_amdgcn_readfirstlane(b1);
    r0 = p0 ? b0 + lane_rank(m0) : -1;
    r1 = p1 ? b1 + lane_rank(m1) : -1;
}

// inclusive prefix sum over the first 32 lanes, or over the wave: row shifts,
// then the row broadcasts
__device__ __forceinline__ int half_wave_incl_scan(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15
    return v;
}

__device__ __forceinline__ int wave_incl_scan(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31
    return v;
}

// Sum over the waves of the workgroup of per-wave values: returns the sum of
// the waves before this one and sets *total.  s_w holds B/64 ints.
template <int B>
__device__ __forceinline__ int waves_before(int wave_total, int *s_w, int *total)
{
    constexpr int NW = B / 64;
    const int w = uni((int)(tid<B>() >> 6));
    if ((tid<B>() & 63) == 0) s_w[w] = wave_total;
    lds_barrier();
    int before = 0, all = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const int t = s_w[i];
        before += i < w ? t : 0;
        all += t;
    }
    *total = all;
    return before;
}

// Exclusive scan over the workgroup.  s_w holds 2 * (B/64) ints; the two
// halves alternate with `phase` so back-to-back calls need one barrier each.
template <int B>
__device__ __forceinline__ int block_excl_scan(int v, int *s_w, int phase, int *total)
{
    const int inc = wave_incl_scan(v);
    const int wt = __builtin_amdgcn_readlane(inc, 63);
    if (B == 64) {
        *total = wt;
        return inc - v;
    }
    return waves_before<B>(wt, s_w + (phase & 1) * (B / 64), total) + inc - v;
}

// Exclusive counts of two predicates over the workgroup (ballots), packed as
// count_a | count_b << 16 like the totals.
template <int B>
__device__ __forceinline__ int block_count2(bool pa, bool pb, int *s_w, int phase, int *total)
{
    const unsigned long long ma = __ballot(pa), mb = __ballot(pb);
    const int mine = lane_rank(ma) | (lane_rank(mb) << 16);
    const int wt = __popcll(ma) | (__popcll(mb) << 16);
    if (B == 64) {
        *total = wt;
        return mine;
    }
    return waves_before<B>(wt, s_w + (phase & 1) * (B / 64), total) + mine;
}

// in-place exclusive scan of a[0..n) in LDS
template <int B>
__device__ __forceinline__ void block_scan_inplace(int *a, int n, int *s_w)
{
    const int chunk = (n + B - 1) / B;
    const int beg = tid<B>() * chunk;
    const int end = beg + chunk < n ? beg + chunk : n;
    int sum = 0;
    for (int i = beg; i < end; ++i) sum += a[i];
    int total;
    int off = block_excl_scan<B>(sum, s_w, 0, &total);
    for (int i = beg; i < end; ++i) {
        int v = a[i];
        a[i] = off;
        off += v;
    }
}

// minimum over lanes lane ^ m, m = 1, 2, 4, 8 (quad permutes for 1 and 2)
__device__ __forceinline__ int lane_xor(int v, int m)
{
    if (m == 1) return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xf, 0xf, false);   // quad_perm [1,0,3,2]
    if (m == 2) return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xf, 0xf, false);   // quad_perm [2,3,0,1]
    return __shfl_xor(v, m);
}

// ---------------------------------------------------------------- LDS layout
// Dynamic LDS of one event workgroup, for a compile-time slot capacity CAP
// (hits per module slot).  The sort scratch (histogram, fill counters, the
// 32-bit sort keys and per-hit bins of events with at most sortcap/2 hits)
// aliases the tracking area, which is filled only after the sort.
//   ring   4 slots x CAP sorted hits (16 B each): traversal index u in slot
//          u mod 4; module t+1 is filled into the slot of t-3 while t is
//          being resolved
//   seeds  the seeds of a step (CAP entries of 10 B): window positions of the
//          three hits, best position of the first following search and its
//          scatter
//   claim  claim words (4 B) of five modules, traversal index u in slot
//          u mod 5, by window position
//   freel  unflagged positions of the seeding stage's doublet module
//   freem  unflagged positions of its middle module
//   tab    coarse phi index of each slot: first position whose phi16 is in
//          bin b or above it
//   own    hit flags of the event, one bit per sorted position, when
//          N <= own_cap (two words of slack behind it)
extern __shared__ __align__(16) char g_lds[];

constexpr int kTab = 256;   // bins of the coarse phi index, at most
constexpr int kSlots = 4;   // ring slots: traversal indices t-2 .. t+1
constexpr int kClaimSlots = 5;   // claim slots: traversal indices t-4 .. t
__host__ __device__ constexpr uint32_t a16(uint32_t v) { return (v + 15u) & ~15u; }
__host__ __device__ constexpr uint32_t lay_seeds(int cap) { return 16u * kSlots * (uint32_t)cap; }
__host__ __device__ constexpr uint32_t lay_freem(int cap) { return lay_seeds(cap) + 10u * (uint32_t)cap; }
__host__ __device__ constexpr uint32_t lay_claim(int cap) { return lay_freem(cap) + 2u * (uint32_t)cap; }
__host__ __device__ constexpr uint32_t lay_freel(int cap) { return lay_claim(cap) + 4u * kClaimSlots * (uint32_t)cap; }
__host__ __device__ constexpr uint32_t lay_tab(int cap) { return lay_freel(cap) + a16(2u * (uint32_t)cap); }
__host__ __device__ constexpr uint32_t lay_own(int cap) { return lay_tab(cap) + 2u * kSlots * kTab; }

// sort bins: 2048 in total, a power of two per module
constexpr int kSortBins = 2048;
__host__ __device__ constexpr uint32_t lds_sort_head() { return a16((kSortBins + 1u) * 4u); }

__host__ __device__ constexpr uint32_t lds_bytes(int cap, int own_cap)
{
    constexpr uint32_t sort = lds_sort_head() + 4u * 1024u;   // keys of 1,024 hits at least
    const uint32_t track = cap > 0 ? lay_own(cap) + a16(4u * (uint32_t)((own_cap + 31) / 32) + 8u) : 0u;
    return sort > track ? sort : track;
}
__host__ __device__ inline int lds_sortcap(int cap, int own_cap)
{
    return (int)((lds_bytes(cap, own_cap) - lds_sort_head()) / 4u);
}

// about a bin per hit: 8 bins per module at least (M <= 64), as many as there
// are at most
__device__ inline int sort_shift(int M, int N)
{
    int bits = 3;
    while (bits < 12 && (M << (bits + 1)) <= kSortBins && (M << bits) < N) ++bits;
    return 16 - bits;
}

template <int CAP>
struct Lay {
    static __device__ __forceinline__ Hit16 *ring(uint32_t lo, int s)
    {
        return reinterpret_cast<Hit16 *>(g_lds + lo) + s * CAP;
    }
    // seeds: CAP words of positions, CAP scatters, CAP halves of positions
    // (seed_words)
    static __device__ __forceinline__ uint32_t *seeds(uint32_t lo)
    {
        return reinterpret_cast<uint32_t *>(g_lds + lo + lay_seeds(CAP));
    }
    static __device__ __forceinline__ uint16_t *seeds16(uint32_t lo)
    {
        return reinterpret_cast<uint16_t *>(g_lds + lo + lay_seeds(CAP) + 8u * CAP);
    }
    static __device__ __forceinline__ uint16_t *freem(uint32_t lo) { return reinterpret_cast<uint16_t *>(g_lds + lo + lay_freem(CAP)); }
    static __device__ __forceinline__ uint32_t *claim(uint32_t lo) { return reinterpret_cast<uint32_t *>(g_lds + lo + lay_claim(CAP)); }
    static __device__ __forceinline__ uint16_t *freel(uint32_t lo) { return reinterpret_cast<uint16_t *>(g_lds + lo + lay_freel(CAP)); }
    static __device__ __forceinline__ uint16_t *tab(uint32_t lo, int s)
    {
        return reinterpret_cast<uint16_t *>(g_lds + lo + lay_tab(CAP)) + s * kTab;
    }
    static __device__ __forceinline__ uint32_t *own(uint32_t lo) { return reinterpret_cast<uint32_t *>(g_lds + lo + lay_own(CAP)); }
};

// Forming tracks of the LDS form are held in registers, one per lane and
// set; as many sets as the slots have hits per lane, so that an event whose
// modules fit runs out of lanes only with more tracks at a step than a module
// may have hits.  (At most four sets, which 64 lanes with 672-hit slots and
// more and 128 with 768 exceed, sent events of more tracks through memory a
// second time: mu = 7.6 x 500 on 64 lanes x 672 slots 1,587 us, now 672; mu in
// U{1..25} x 300 on 128 x 768 1,560, now 642.)
template <int B, int CAP>
__host__ __device__ constexpr int track_sets()
{
    return CAP <= B ? 1 : (CAP + B - 1) / B;
}

// static LDS shared by the stages of one event
template <int B>
struct Shared {
    int mo[SBT_MAX_MODULES + 1];
    int cnt[4];          // records, list[0], list[1], final
    int status;
    int e;
    int maxmod;          // hits of the event's largest module
    alignas(16) int ctl[4];   // LDS form: seeds of a step by its parity (0, 1), a tie of claims, final records (read as one int4)
    int scan[2 * (B / 64)];
    union alignas(16) {
        uint8_t mtab[(SBT_MAX_EVENT_HITS + 64) / 64];   // module of every 64th hit (sort)
        // LDS form: by traversal index the first sorted position, hits and
        // nominal z; in w, by free_at, the free track slots of the waves
        int4 mt[SBT_MAX_MODULES];
    };
};

// Events of 64 lanes run one per wave, up to this many in a workgroup; each
// takes a region of the dynamic LDS: its Shared block, then its layout.
constexpr int kMaxEventsPerBlock = 16;
template <int B>
__host__ __device__ constexpr uint32_t shared_block_bytes()
{
    return a16((uint32_t)sizeof(Shared<B>));
}
template <int B>
__host__ __device__ constexpr uint32_t event_region_bytes(int cap, int own_cap)
{
    return shared_block_bytes<B>() + lds_bytes(cap, own_cap);
}

// LDS of a compute unit, and the most dynamic LDS a workgroup may ask for
constexpr uint32_t kCuLds = 160 * 1024, kMaxDynLds = kCuLds - 1024;

// Lanes of the widest workgroup that runs events of B lanes: 64-lane events
// as many to a workgroup as have room in its LDS.
template <int B, int CAP>
constexpr int max_block_lanes()
{
    if (B > 64) return B;
    const int fit = (int)(kMaxDynLds / event_region_bytes<B>(CAP, 0));
    return 64 * (fit < kMaxEventsPerBlock ? fit : kMaxEventsPerBlock);
}

// Waves per SIMD that a persistent kernel leaves registers for: four, five
// with 256 lanes (five workgroups with 256-hit slots on a CU), and no more than
// the LDS lets run, so that the sets of forming tracks stay in registers (with
// four and five for all of them, 64 to 256 lanes spilled 8 to 133).
template <int B, int CAP>
constexpr int simd_waves()
{
    constexpr int most = B == 256 ? 5 : 4;
    const int groups = (int)(kCuLds / event_region_bytes<B>(CAP, 0));
    const int waves = (groups * (B / 64) + 3) / 4;
    return waves < most ? waves : most;
}

// Where the free track slots of a wave stand in Shared::mt, for the sets
// 2 h (low half) and 2 h + 1 (high half), by the parity of the step.
template <int B, int CAP>
constexpr int free_words()
{
    constexpr int words = (track_sets<B, CAP>() + 1) / 2;
    static_assert(2 * words * (B / 64) <= SBT_MAX_MODULES, "free slots beside the module table");
    return words;
}
template <int B, int CAP>
__device__ __forceinline__ int &free_at(Shared<B> &S, int parity, int h, int wave)
{
    return S.mt[(parity * free_words<B, CAP>() + h) * (B / 64) + wave].w;
}

// per-event views of the workspace: pointers are derived on use from the
// base, the capacity H and the event's hit offset hb
struct Ev {
    char *base;
    uint32_t H, E;
    int e, hb, N;
    uint32_t lo;   // byte offset of the event's region in the workgroup's dynamic LDS
    template <class T>
    __device__ __forceinline__ T *arr(uint32_t off, uint32_t elem) const
    {
        return reinterpret_cast<T *>(base + (uint64_t)H * off + (uint64_t)(uint32_t)hb * elem);
    }
    __device__ __forceinline__ Rec *rec() const { return arr<Rec>(kOffRec, 32); }
    __device__ __forceinline__ uint4 *fin() const { return reinterpret_cast<uint4 *>(rec()); }   // final records of the LDS form
    __device__ __forceinline__ uint16_t *sid() const { return list(kListFRank); }                // its ids by sorted position
    __device__ __forceinline__ Hit16 *hs() const { return arr<Hit16>(kOffHs, 16); }
    __device__ __forceinline__ RecAux *aux() const { return arr<RecAux>(kOffAux, 16); }
    __device__ __forceinline__ unsigned long long *claim() const { return arr<unsigned long long>(kOffClaim, 8); }
    __device__ __forceinline__ uint32_t *keys() const { return arr<uint32_t>(kOffKeys, 4); }
    __device__ __forceinline__ uint16_t *link() const { return arr<uint16_t>(kOffLink, 4); }   // [2i] prev, [2i+1] key -> record
    __device__ __forceinline__ int32_t *st_toff() const { return arr<int32_t>(kOffToff, 4); }
    __device__ __forceinline__ uint16_t *st_hits() const { return arr<uint16_t>(kOffStHits, 2); }
    __device__ __forceinline__ uint16_t *list(int k) const
    {
        return reinterpret_cast<uint16_t *>(base + (uint64_t)H * (kOffLists + 2u * k) + (uint64_t)(uint32_t)hb * 2);
    }
    __device__ __forceinline__ uint32_t *own() const
    {
        return reinterpret_cast<uint32_t *>(base + ws_owner(H)) + ((uint32_t)hb >> 5) + e;
    }
    __device__ __forceinline__ EvInfo &info() const
    {
        return reinterpret_cast<EvInfo *>(base + ws_ev(H, E))[e];
    }
};

__device__ __forceinline__ Ev event_view(const Work &W, int e, int hb, int N, uint32_t lo = 0)
{
    Ev v;
    v.base = opq_global(W.base);
    v.H = opq(W.H);
    v.E = W.E;
    v.e = e;
    v.hb = hb;
    v.N = N;
    v.lo = lo;
    return v;
}

// the view with its base hidden from the optimiser (see opq)
__device__ __forceinline__ Ev fresh(const Ev &v)
{
    Ev w = v;
    w.base = opq_global(v.base);
    w.H = opq(v.H);
    return w;
}

// ---------------------------------------------------------------- validation
// Loads the event-local module offsets into LDS and checks the offsets.
template <int B>
__device__ __forceinline__ int load_event(const sbt_params &P, const HitsArgs &H, int e, Shared<B> &S,
                          int *hb_out, int *n_out)
{
    const int M = P.n_modules;
    int lo = H.eo[e], hi = H.eo[e + 1];
    if (tid<B>() == 0) {
        S.status = 0;
        S.maxmod = 0;
    }
    ev_sync<B>();
    unsigned st = 0;
    if (lo < 0 || hi > H.n_hits || hi < lo) st = SBT_EV_BAD_OFFSETS;
    else if (hi - lo > SBT_MAX_EVENT_HITS) st = SBT_EV_TOO_LARGE;
    else if (P.max_event_hits > 0 && hi - lo > P.max_event_hits) st = SBT_EV_CUT;
    if (st == 0) {
        const long long base = (long long)e * M;
        for (int k = tid<B>(); k <= M; k += B) {
            int v = H.mo[base + k];
            S.mo[k] = v - lo;
            bool bad = (k == 0 && v != lo) || (k == M && v != hi) || v < lo || v > hi;
            if (k > 0 && H.mo[base + k - 1] > v) bad = true;
            if (bad) atomicOr(&S.status, (int)SBT_EV_BAD_OFFSETS);
            if (k < M) atomicMax(&S.maxmod, H.mo[base + k + 1] - v);
        }
    } else if (tid<B>() == 0) {
        S.status = (int)st;
    }
    ev_sync<B>();
    *hb_out = uni(lo);
    *n_out = uni(hi - lo);
    return uni(S.status);
}

// ---------------------------------------------------------------- hit coordinates
// Coordinates of event-local hit i, from binary32 arrays or widened exactly
// from the binary16 array-of-structures form.
__device__ __forceinline__ float half_bits_to_float(uint32_t b)
{
    return (float)__builtin_bit_cast(_Float16, (uint16_t)(b & 0xFFFFu));
}

struct HitSrc {
    const float *x, *y, *z;
    const uint2 *h16;
    __device__ __forceinline__ void xy(int i, float &px, float &py) const
    {
        if (h16) {
            const uint2 w = at(h16, i);
            px = half_bits_to_float(w.x);
            py = half_bits_to_float(w.x >> 16);
        } else {
            px = at(x, i);
            py = at(y, i);
        }
    }
    __device__ __forceinline__ void xyz(int i, float &px, float &py, float &pz) const
    {
        if (h16) {
            const uint2 w = at(h16, i);
            px = half_bits_to_float(w.x);
            py = half_bits_to_float(w.x >> 16);
            pz = half_bits_to_float(w.y);
        } else {
            px = at(x, i);
            py = at(y, i);
            pz = at(z, i);
        }
    }
};

__device__ __forceinline__ HitSrc hit_src(const HitsArgs &H, int hb)
{
    HitSrc s;
    s.h16 = H.h16 ? H.h16 + hb : nullptr;
    s.x = H.h16 ? nullptr : H.x + hb;
    s.y = H.h16 ? nullptr : H.y + hb;
    s.z = H.h16 ? nullptr : H.z + hb;
    return s;
}

// ---------------------------------------------------------------- sort by phi
// Counting sort on (module, top bits of phi16) into buckets of 32-bit keys
// phi16 << 16 | id, then each key's rank inside its bucket by counting the
// smaller keys of the bucket; ties in phi16 fall to the lower id because the
// id is the key's low half.  Three forms by event size against the LDS key
// capacity sortcap: keys and per-hit bins in LDS (2N <= sortcap); keys in
// LDS with the bins recomputed (N <= sortcap); both in memory.
// module of hit i from the module of its 64-hit chunk and a short forward scan
__device__ __forceinline__ int sort_bin(const int *mo, const uint8_t *mtab, int i, uint16_t q, int bpm, int shift)
{
    int m = mtab[i >> 6];
    while (mo[m + 1] <= i) ++m;
    return m * bpm + (q >> shift);
}

constexpr int kSortChunk = 8;   // hits of a lane whose coordinates are loaded together
constexpr int kSortBatch = 4;   // hits of a lane on their way through the LDS together

// Keys into their bins: a bin's start is its cursor, and its end afterwards.
template <int B, int J>
__device__ __forceinline__ void sort_place(const HitSrc &src, const Shared<B> &S, int *hist, uint32_t *lkeys, int N,
                                           int form, int bpm, int shift)
{
    for (int i0 = tid<B>(); i0 < N; i0 += J * B) {
        uint32_t tb[J];
        if (form == 0) {
#pragma unroll
            for (int j = 0; j < J; ++j) tb[j] = lkeys[N + min(i0 + j * B, N - 1)];
        } else {
            float px[J], py[J];
#pragma unroll
            for (int j = 0; j < J; ++j) src.xy(min(i0 + j * B, N - 1), px[j], py[j]);
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const uint16_t qi = phi16(px[j], py[j]);
                tb[j] = (uint32_t)qi |
                        ((uint32_t)sort_bin(S.mo, S.mtab, min(i0 + j * B, N - 1), qi, bpm, shift) << 16);
            }
        }
        int at0[J];
#pragma unroll
        for (int j = 0; j < J; ++j) at0[j] = i0 + j * B < N ? atomicAdd(&hist[tb[j] >> 16], 1) : 0;
#pragma unroll
        for (int j = 0; j < J; ++j)
            if (i0 + j * B < N) lkeys[at0[j]] = (tb[j] << 16) | (uint32_t)(i0 + j * B);
    }
}

// A key's rank in its bin, by the smaller keys there, and the sorted hit.
template <int B, int J>
__device__ __forceinline__ void sort_rank(const Ev &v, const HitSrc &src, const Shared<B> &S, const int *hist,
                                          const uint32_t *lkeys, int N, int bpm, int shift)
{
    for (int s0 = tid<B>(); s0 < N; s0 += J * B) {
        uint32_t key[J];
        Hit16 h[J];
        int rank[J], m[J], hi[J];
#pragma unroll
        for (int j = 0; j < J; ++j) key[j] = lkeys[min(s0 + j * B, N - 1)];
#pragma unroll
        for (int j = 0; j < J; ++j) src.xyz((int)(key[j] & 0xFFFFu), h[j].x, h[j].y, h[j].z);
        bool more = false;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            // a slot lies in the module of its hit
            const int bin = sort_bin(S.mo, S.mtab, min(s0 + j * B, N - 1), (uint16_t)(key[j] >> 16), bpm, shift);
            m[j] = bin > 0 ? hist[bin - 1] : 0;
            hi[j] = hist[bin];
            rank[j] = m[j];
            more = more || m[j] < hi[j];
        }
        while (more) {
            more = false;
            uint32_t o[J];
#pragma unroll
            for (int j = 0; j < J; ++j) o[j] = lkeys[min(m[j], N - 1)];
#pragma unroll
            for (int j = 0; j < J; ++j) {
                rank[j] += m[j] < hi[j] && o[j] < key[j];
                ++m[j];
                more = more || m[j] < hi[j];
            }
        }
#pragma unroll
        for (int j = 0; j < J; ++j)
            if (s0 + j * B < N) {
                h[j].qid = (key[j] >> 16) | (key[j] << 16);
                at(v.hs(), rank[j]) = h[j];
            }
    }
}

// Every pass is a chain of LDS round trips per hit (bin, start, cursor, key;
// key, bin, range, ranks), so a lane takes kSortBatch hits through it side by
// side, there is about a bin per hit, and one array holds counts, cursors and ends of
// the bins.  Against one hit at a time and 32 bins a module: the largest mu = 7.6
// event (9,786 hits) 112 k -> 78 k cycles, mu in U{1..25} x 10,000 3,947 -> 3,864 us.
template <int B>
__device__ __forceinline__ void stage_sort(const sbt_params &PP, const HitsArgs &H, const Ev &v0, Shared<B> &S, int sortcap)
{
    const Ev v = fresh(v0);
    const int M = fresh(PP).M, N = v.N;
    const int shift = sort_shift(M, N);
    const int bpm = 1 << (16 - shift);
    const int nb = M * bpm;
    int *hist = reinterpret_cast<int *>(g_lds + v.lo);   // counts, then starts, then ends of the bins
    uint32_t *lkeys = reinterpret_cast<uint32_t *>(g_lds + v.lo + lds_sort_head());
    const int form = 2 * N <= sortcap ? 0 : (N <= sortcap ? 1 : 2);
    for (int i = tid<B>(); i <= nb; i += B) hist[i] = 0;
    for (int c = tid<B>(); c < (N + 63) / 64; c += B) S.mtab[c] = (uint8_t)module_of(S.mo, M, c * 64);
    ev_sync<B>();
    const HitSrc src = hit_src(H, v.hb);
    // memory form: bins in the claim words (not yet in use)
    uint32_t *bins_m = reinterpret_cast<uint32_t *>(v.claim());
    // the coordinates of a lane's next kSortChunk hits are loaded together
    for (int i0 = tid<B>(); i0 < N; i0 += kSortChunk * B) {
        float px[kSortChunk], py[kSortChunk];
#pragma unroll
        for (int j = 0; j < kSortChunk; ++j)
            if (i0 + j * B < N) src.xy(i0 + j * B, px[j], py[j]);
#pragma unroll
        for (int j = 0; j < kSortChunk; ++j) {
            const int i = i0 + j * B;
            if (i >= N) break;
            const uint16_t qi = phi16(px[j], py[j]);
            const int bin = sort_bin(S.mo, S.mtab, i, qi, bpm, shift);
            const uint32_t tb = (uint32_t)qi | ((uint32_t)bin << 16);
            if (form == 0) lkeys[N + i] = tb;
            else if (form == 2) at(bins_m, i) = tb;
            atomicAdd(&hist[bin], 1);
        }
    }
    ev_sync<B>();
    block_scan_inplace<B>(hist, nb + 1, S.scan);
    ev_sync<B>();
    // separate LDS and memory branches keep each access in its address space
    if (form == 2) {
        for (int i = tid<B>(); i < N; i += B) {
            const uint32_t tb = at(bins_m, i);
            at(v.keys(), atomicAdd(&hist[tb >> 16], 1)) = (tb << 16) | (uint32_t)i;
        }
    } else {
        if (N <= B) sort_place<B, 1>(src, S, hist, lkeys, N, form, bpm, shift);
        else sort_place<B, kSortBatch>(src, S, hist, lkeys, N, form, bpm, shift);
    }
    ev_sync<B>();
    if (form == 2) {
        for (int s = tid<B>(); s < N; s += B) {
            const uint32_t key = at(v.keys(), s);
            const int i = (int)(key & 0xFFFFu);
            const int bin = (int)(at(bins_m, i) >> 16);
            const int lo = bin > 0 ? hist[bin - 1] : 0, hi = hist[bin];
            int rank = lo;
            for (int m = lo; m < hi; ++m) rank += at(v.keys(), m) < key;
            Hit16 h;
            src.xyz(i, h.x, h.y, h.z);
            h.qid = (key >> 16) | (key << 16);
            at(v.hs(), rank) = h;
        }
    } else {
        if (N <= B) sort_rank<B, 1>(v, src, S, hist, lkeys, N, bpm, shift);
        else sort_rank<B, kSortBatch>(v, src, S, hist, lkeys, N, bpm, shift);
    }
    ev_sync<B>();
}

// ---------------------------------------------------------------- module windows
// An event whose modules all fit the LDS slots (and whose hit flags fit the
// LDS bitmap) runs the LDS form of the tracking stages: traversal index u
// lives in ring slot u mod 4 and every window access is an LDS access.  Any
// other event runs the memory form, which reads the sorted hits in memory
// directly.  Both compute the same thing.  The LDS form names a hit by its
// sorted position, the memory form by its id.
struct Win {
    const Hit16 *h;
    int n;
};

__device__ __forceinline__ uint16_t q_of(const Hit16 &h) { return (uint16_t)(h.qid & 0xFFFFu); }
__device__ __forceinline__ uint16_t id_of(const Hit16 &h) { return (uint16_t)(h.qid >> 16); }
__device__ __forceinline__ uint16_t win_q(const Win &w, int p) { return (uint16_t)(at(w.h, p).qid & 0xFFFFu); }
__device__ __forceinline__ uint16_t win_id(const Win &w, int p) { return (uint16_t)(at(w.h, p).qid >> 16); }

// first position of the window whose phi16 is >= v
__device__ __forceinline__ int win_lower_bound(const Win &w, uint16_t v)
{
    int lo = 0, hi = w.n;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (win_q(w, mid) < v) lo = mid + 1; else hi = mid;
    }
    return lo;
}

template <int B>
__device__ __forceinline__ Win window(const Prm &P, const Shared<B> &S, const Ev &v, int u)
{
    Win w;
    const int k = kmod(P, u);
    const int g0 = uni(S.mo[k]);
    w.n = uni(S.mo[k + 1]) - g0;
    w.h = v.hs() + g0;
    return w;
}

// ---------------------------------------------------------------- seeding
// Tracklet fit of a seed, hits in traversal order (Section 3, "Tracklet
// filter"): chi2 = ((v.x)^2 + (v.y)^2) / (v.v) with v = (z2-z1, z0-z2, z1-z0)
// orthogonal to (1,1,1) and to z
__device__ __forceinline__ float seed_chi2(const Hit16 &h0, const Hit16 &h1, const Hit16 &h2)
{
    const float v0 = h2.z - h1.z, v1 = h0.z - h2.z, v2 = h1.z - h0.z;
    const float ssx = ((v0 * h0.x) + (v1 * h1.x)) + (v2 * h2.x);
    const float ssy = ((v0 * h0.y) + (v1 * h1.y)) + (v2 * h2.y);
    const float n2 = ((v0 * v0) + (v1 * v1)) + (v2 * v2);
    return ((ssx * ssx) + (ssy * ssy)) / n2;
}

// The pendulum search visits the doublet module's phi-sorted positions in
// the order s0, s0-1, s0+1, s0-2, s0+2, ... (wrapping, at most n visits) and
// keeps the first K unflagged ones.  Here the unflagged positions are first
// compacted in order; the K kept ones are then the K of smallest visit rank
// (offset o >= 0 -> 2o, o < 0 -> -2o-1), found by merging the walks up and
// down from s0 through the compacted list.  Returns the position of the
// c-th kept partner, or -1.
__device__ __forceinline__ int pendulum_pick(const uint16_t *F, int nf, int j, int s0, int na, int hu, int hd, int c)
{
    int su = 0, sd = 0, pos = -1;
    for (int step = 0; step <= c; ++step) {
        int vu = 0x7fffffff, vd = 0x7fffffff, pu = 0, pd = 0;
        if (su < nf) {
            int ix = j + su;
            if (ix >= nf) ix -= nf;
            pu = at(F, ix);
            int o = pu - s0;
            if (o < 0) o += na;
            if (o <= hu) vu = 2 * o;
        }
        if (sd < nf) {
            int ix = j - 1 - sd;
            if (ix < 0) ix += nf;
            pd = at(F, ix);
            int o = s0 - pd;
            if (o < 0) o += na;
            if (o >= 1 && o <= hd) vd = 2 * o - 1;
        }
        if (vu == 0x7fffffff && vd == 0x7fffffff) return -1;
        if (vd == 0x7fffffff || vu < vd) { pos = pu; ++su; }
        else { pos = pd; ++sd; }
    }
    return pos;
}

// One of the K = 4 picks for lane c = 0..3 of a middle hit, a different one
// for each lane, or -1: which lane gets which does not matter, as the lanes'
// doublets meet in a minimum.  The unflagged positions upwards from s0 and
// those downwards below it are two lists of ascending visit ranks (2o and 2o -
// 1 for an offset o); the four smallest of two ascending lists of four are
// min(up[c], down[3 - c]), so a lane loads those two and needs no other lane.
// (Exchanging the eight ranks and merging them to the c-th smallest took some
// 60 instructions more on the step's chain: mu = 7.6 x 1,000 279 us, now 274;
// mu in U{1..25} x 1,000 392, now 383; one event of 500 hits 71.6, now 70.0.)
__device__ __forceinline__ int pendulum_quad(const uint16_t *F, int nf, int j, int s0, int na, int hu, int hd, int c)
{
    constexpr int kInf = 0x7fffffff;
    int ru = kInf, rd = kInf, pu = 0, pd = 0;
    if (c < nf) {
        int iu = j + c;
        if (iu >= nf) iu -= nf;
        pu = at(F, iu);
        int o = pu - s0;
        if (o < 0) o += na;
        if (o <= hu) ru = 2 * o;
    }
    if (3 - c < nf) {
        int id = j - 4 + c;
        if (id < 0) id += nf;
        pd = at(F, id);
        int o = s0 - pd;
        if (o < 0) o += na;
        if (o >= 1 && o <= hd) rd = 2 * o - 1;
    }
    return min(ru, rd) == kInf ? -1 : ru < rd ? pu : pd;
}


// ================================================================ LDS form
// One step costs two barriers.  R(t): every forming track tests the claims of
// its search into t and extends, waits or ends; the next module enters the
// ring.  S(t): the seeds of t and their first search, and the kept tracks'
// searches, all into t+1.  What bounds it is the dependent chain of a step
// (LDS round trips, correctly rounded divisions, window walks), run 24 times
// per event, and the instructions issued for it, so
//   - a forming track stays in the registers of one lane from its seed to its
//     end, and its step touches no memory but the previous-hit link it leaves
//     behind; new seeds go to the lowest free lanes, so that few waves carry
//     tracks and the others seed;
//   - hits are named by sorted position, so the flags of a module are a run of
//     bits and every wave that seeds takes the unflagged positions from a few
//     words by itself, without a barrier;
//   - the claims on a bare seed's hits are LDS words like those on the best
//     hits (five modules of them), and the sorted hits of the module after
//     the next are in registers a step before they are needed.
// Measured against the form before it (tracks as 32-byte records in memory,
// hits named by id, four barriers a step; microseconds a call): one event of
// 500 hits 121 -> 81, one mu = 7.6 event 181 -> 124, mu = 7.6 x 1,000 452 ->
// 350, mu in U{1..25} x 10,000 5,796 -> 4,142.  With the shared lists of
// unflagged positions, four lanes per middle hit, the bound as first best key
// and walks over several hits at a time, partners without an exchange, and
// fewer launches around it, the same calls take 71, 117, 277 and 3,220.

struct LWin {
    const Hit16 *h;
    const uint16_t *tab;
    int n, sh;      // hits; phi16 >> sh is the coarse index bin
};

// about one bin per hit: 32 to kTab bins
__device__ __forceinline__ int tab_shift(int n) { return n > 192 ? 8 : n > 96 ? 9 : n > 48 ? 10 : 11; }

template <int CAP>
__device__ __forceinline__ LWin lds_window(uint32_t lo, int u, int n)
{
    LWin w;
    w.h = Lay<CAP>::ring(lo, u & (kSlots - 1));
    w.tab = Lay<CAP>::tab(lo, u & (kSlots - 1));
    w.n = n;
    w.sh = tab_shift(n);
    return w;
}

// forming track: its last two hits, the seed's hits and the last one by
// sorted position, and the result of its search
struct Trk {
    float xa, ya, za, xb, yb, zb;
    uint32_t k0;     // key | h0 << 16
    uint32_t h12;    // h1 | h2 << 16
    uint32_t lst;    // last | hits << 16 | traversal index of the last << 24; 0: no track
    uint32_t pb;     // window position of the best hit, or kNoPos
    float bsc;       // its scatter
};
// A seed's positions (below 2,047) in the seeds table: pos0 | pos1 << 11 | pos2
// << 22 (its low ten bits) and pos2 >> 10 | best << 1.
constexpr uint32_t kNoPos = 0x7FFu;

// final record of the LDS form: key | h0 << 16, h1 | h2 << 16, last | hits << 16
typedef uint4 Fin;

// Claim word of the LDS form: 63 - stage above the leading 26 bits of the
// score.  As in claim_key, a word left from an earlier stage is larger than
// any of a later one.  Of two claims of one stage that agree in those bits on
// one word the second meets its own value there; the resolution then settles
// that stage over 64-bit words in memory (claim_key).
__device__ __forceinline__ uint32_t claim32(float score, int stage)
{
    return ((uint32_t)(63 - stage) << 26) | (__float_as_uint(score) >> 5);
}

// Hits that a walk takes at a time.  Its loop's own instructions (the masks of
// who is done, the count, the branch) and an LDS round trip are shared by them,
// and a walk meets up to one less than that many hits behind its window.  Two
// instead of one take mu = 7.6 x 1,000 from 291 to 284 us and mu = 30 x 400
// from 538 to 501; three 282 and 494, four 282 and 498, six 290 and 504.
// Small slots have short windows, and the instance held to 80 registers
// spills with more (mu = 7.6 x 4,000: two 862, three 862, four 886).
constexpr int walk_unroll(int cap) { return cap >= 672 ? 3 : 2; }

// Walks the window [lo, lo + span] of phi16 from the start of lo's bin on
// `stride` lanes (this one the k-th), U positions at a time, and calls
// hit(h, p, in) for the positions this lane meets, in or out of the window:
// positions of the bin below lo come first (their distance to lo is within a
// bin of a full turn), then the window, then some beyond it.  A position may
// be met twice where the walk closes the circle; the callers take minima.  The lanes of a
// wave walk together until the last one is done, with masks for branches: what a walk
// costs is the instructions of its longest window.
template <int U, class F>
__device__ __forceinline__ void walk(const LWin &w, uint32_t lo, uint32_t span, int k, int stride, F &&hit)
{
    uint32_t p = at(w.tab, lo >> w.sh) + (uint32_t)k;
    p = min(p, p - (uint32_t)w.n);   // p - n is huge while p < n
    unsigned long long live = __ballot(k < w.n);
    p = k < w.n ? p : 0u;
    const uint32_t below = 0x10000u - (1u << w.sh);
    // q + step - n stays under n: where the lanes already cover the module, no step
    const uint32_t step = w.n > stride ? (uint32_t)stride : 0u;
    for (int left = uni(w.n); left > 0; left -= U * stride) {
        uint32_t q[U];
        Hit16 h[U];
        q[0] = p;
#pragma unroll
        for (int i = 1; i < U; ++i) {
            const uint32_t x = q[i - 1] + step;
            q[i] = min(x, x - (uint32_t)w.n);
        }
#pragma unroll
        for (int i = 0; i < U; ++i) h[i] = at(w.h, q[i]);
#pragma unroll
        for (int i = 0; i < U; ++i) hit(h[i], (int)q[i], ((h[i].qid - lo) & 0xFFFFu) <= span);
        const uint32_t d = (h[U - 1].qid - lo) & 0xFFFFu;
        live &= __ballot(d <= span) | __ballot(d >= below);
        if (live == 0ull) break;
        const uint32_t x = q[U - 1] + step;
        p = min(x, x - (uint32_t)w.n);
    }
}

// The smallest key that is not under a strict bound on the scatter, where keys
// are (scatter bits, ids) and scatters are >= +0: a search that starts from it
// takes only keys under the bound (none where the bound is not positive; a
// NaN is above every bound).
__device__ __forceinline__ unsigned long long bound_key(float bound)
{
    return bound > 0.0f ? (unsigned long long)__float_as_uint(bound) << 32 : 0ull;
}

// Search of a track into the window: best hit by (scatter, id) under the bound
// in bk, as one word that orders like the pair, and its position.
template <int U>
__device__ __forceinline__ void follow_walk(const LWin &w, float xb, float yb, float zb, float tx, float ty, float Zn,
                                            int Wf, int k, int stride, unsigned long long &bk, uint32_t &bp)
{
    const float dzc = Zn - zb;
    const uint32_t lo = (uint32_t)(phi16(xb + tx * dzc, yb + ty * dzc) - Wf) & 0xFFFFu;
    walk<U>(w, lo, 2u * (uint32_t)Wf, k, stride, [&](const Hit16 &h, int p, bool in) {
        const float dz = h.z - zb;
        const float dx = (xb + tx * dz) - h.x;
        const float dy = (yb + ty * dz) - h.y;
        const float sc = (dx * dx) + (dy * dy);
        const unsigned long long key = ((unsigned long long)__float_as_uint(sc) << 32) | (h.qid >> 16);
        const bool better = in && key < bk;
        bk = better ? key : bk;
        bp = better ? (uint32_t)p : bp;
    });
}

// Scalars of step t, by module: index i is traversal index t - 4 + i.
struct Step {
    int t;
    int g[7], n[7];      // first sorted position, hits
    int c[5];            // claim slot offsets (index 5, t + 1, shares that of t - 4)
    float Zc, Zn, Zx;    // nominal z of t, t + 1 and t + 2
};

// unflagged positions [64 w, 64 w + 64) of a module of n hits whose first
// sorted position is g
// (n > 0; the word is empty past the module's last)
__device__ __forceinline__ unsigned long long free_word(const uint32_t *own, int g, int n, int w)
{
    const int x = min(w, (n - 1) >> 6);
    const uint32_t b = (uint32_t)(g + 64 * x);
    const uint32_t r0 = at(own, b >> 5), r1 = at(own, (b >> 5) + 1u), r2 = at(own, (b >> 5) + 2u);
    const uint32_t lo = __builtin_amdgcn_alignbit(r1, r0, b & 31u), hi = __builtin_amdgcn_alignbit(r2, r1, b & 31u);
    const unsigned long long m = ~(((unsigned long long)hi << 32) | lo);
    const int rem = n - 64 * w;
    const unsigned long long in = rem >= 64 ? ~0ull : (1ull << (rem & 63)) - 1ull;
    return rem <= 0 ? 0ull : m & in;
}

__device__ __forceinline__ unsigned long long read_lane64(unsigned long long v, int l)
{
    const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l);
    return ((unsigned long long)b << 32) | a;
}

// minimum of (key, pos) over the G lanes of a group (KQ = 4: by quad permutes;
// every lane gets it)
template <int KQ>
__device__ __forceinline__ void group_min(unsigned long long &key, uint32_t &pos, int G)
{
    for (int m = 1; m < (KQ ? KQ : G); m <<= 1) {
        const uint32_t olo = (uint32_t)lane_xor((int)(uint32_t)key, m);
        const uint32_t ohi = (uint32_t)lane_xor((int)(uint32_t)(key >> 32), m);
        const uint32_t op = (uint32_t)lane_xor((int)pos, m);
        const unsigned long long o = ((unsigned long long)ohi << 32) | olo;
        const bool less = o < key;
        key = less ? o : key;
        pos = less ? op : pos;
    }
}

// The unflagged positions of a step's doublet and middle modules: lane w
// holds word w of A and the unflagged positions before it.
struct Free {
    unsigned long long a;
    int ex;
    int na, nb;    // unflagged positions of A, of Bm
};

// Seeding of step t (Section 3) on the waves from the last one down: modules
// A = t-2, Bm = t-1, C = t; work items are (unflagged middle hit, partner
// rank c), the K doublets of a middle hit on K adjacent lanes where K is a
// power of two up to 16 (KQ = 4: known at compile time), all on one lane
// otherwise.  A new seed's search into t+1 runs on the lanes that made it;
// seed and result go to the seeds table.  (More lanes for a middle hit, two or
// four to a doublet's walk, shorten the chain but are more instructions, which
// the SIMDs have no room for where a CU holds two events: with walks of one
// hit at a time sixteen lanes took 317 us for mu = 7.6 x 1,000, eight 294,
// these four 297, and 1,703, 1,618 and 1,606 for mu in U{1..25} x 4,000.)
template <int B, int CAP, int KQ, bool kCand>
__device__ __forceinline__ void seed_pass(const Prm &P, uint32_t lo, const uint32_t *cand, const Step &st,
                                          Shared<B> &S, const Free &fr, bool more, bool gc)
{
    constexpr int NW = B / 64;
    const int lane = (int)(tid<B>() & 63);
    const int sw = NW - 1 - uni((int)(tid<B>() >> 6));
    const int K = KQ ? KQ : P.K;
    const int G = KQ == 4 ? 4 : (K == 1 || K == 2 || K == 4 || K == 8 || K == 16) ? K : 1;
    const int per_lane = KQ == 4 ? 1 : (G == 1 ? K : 1);
    const int items = fr.nb * G;
    if (sw * 64 >= items) return;

    // the seeding waves carry the longest dependency chain of the step
    __builtin_amdgcn_s_setprio(2);
    const int na = st.n[2], nf = fr.na;
    const int Ws = P.Ws;
    const unsigned long long none = bound_key(P.Ss), none_f = bound_key(P.Sf);
    const uint16_t *F = Lay<CAP>::freel(lo), *FM = Lay<CAP>::freem(lo);
    const LWin wa = lds_window<CAP>(lo, st.t - 2, na);
    const LWin wc = lds_window<CAP>(lo, st.t, st.n[4]);
    const Hit16 *hb = Lay<CAP>::ring(lo, (st.t - 1) & (kSlots - 1));
    const int hd = na >> 1, hu = na - hd - 1;   // offsets visited: [-hd, hu]

    for (int base = sw * 64; base < items; base += B) {
        const int g = base + lane;
        const bool on = g < items;
        const int i = KQ == 4 ? g >> 2 : g / G;
        const int c = KQ == 4 ? g & 3 : g - i * G;   // partner rank: the lane of the group
        const int p1 = on ? at(FM, (uint32_t)i) : 0;
        const Hit16 h1 = at(hb, (uint32_t)p1);
        // pendulum start: the first position of A whose phi16 is not below the middle hit's
        int s0 = 0;
        if (kCand) {
            if (on) s0 = (int)at(cand, (uint32_t)(st.g[3] + p1));
        } else if (KQ == 4) {
            // the group's lanes test as many positions at a time
            const uint32_t q1 = q_of(h1);
            s0 = at(wa.tab, q1 >> wa.sh);
            for (;;) {
                const int x = s0 + (lane & (G - 1));
                const bool less = x < na && q_of(at(wa.h, (uint32_t)(x < na ? x : 0))) < q1;
                const uint32_t m = (uint32_t)(__ballot(less) >> (lane & (64 - G))) & ((1u << G) - 1u);
                s0 += __popc(m);
                if (__ballot(m == (1u << G) - 1u) == 0ull) break;
            }
            if (s0 == na) s0 = 0;
        } else if (on) {
            const uint32_t q1 = q_of(h1);
            s0 = at(wa.tab, q1 >> wa.sh);
            while (s0 < na && q_of(at(wa.h, (uint32_t)s0)) < q1) ++s0;
            if (s0 == na) s0 = 0;
        }
        // unflagged positions below s0: the index in F of the first one at or
        // above it (words from the lane that holds them, every lane active)
        const int sl = s0 >> 6;
        const uint32_t alo = (uint32_t)__shfl((int)(uint32_t)fr.a, sl), ahi = (uint32_t)__shfl((int)(uint32_t)(fr.a >> 32), sl);
        const unsigned long long aw = ((unsigned long long)ahi << 32) | alo;
        const int j = (__shfl(fr.ex, sl) & 0xFFFF) + __popcll(aw & ((1ull << (s0 & 63)) - 1ull));

        unsigned long long bkey = none;
        uint32_t bp0 = 0, bpos = kNoPos;   // positions of the best triplet's first and third hits
        for (int cc = 0; cc < per_lane; ++cc) {
            const int pos0 = !on ? -1 : KQ == 4 ? pendulum_quad(F, nf, j, s0, na, hu, hd, c)
                                                : pendulum_pick(F, nf, j, s0, na, hu, hd, c + cc);
            if (pos0 < 0) break;
            // best third hit of the doublet: the key orders like the comparison
            // (found, scatter, id0, id2); the packed positions are pos2 | pos0 << 16.  Hits of
            // C that are flagged hold no coordinate and fail the comparison.
            const Hit16 h0 = at(wa.h, (uint32_t)pos0);
            const uint32_t id0 = h0.qid >> 16;
            const float d01 = h1.z - h0.z;
            const float tx = (h1.x - h0.x) / d01;
            const float ty = (h1.y - h0.y) / d01;
            const float dzc = st.Zc - h1.z;
            const uint32_t from = (uint32_t)(phi16(h1.x + tx * dzc, h1.y + ty * dzc) - Ws) & 0xFFFFu;
            walk<walk_unroll(CAP)>(wc, from, 2u * (uint32_t)Ws, 0, 1,
                 [&](const Hit16 &h2, int p, bool in) {
                     const float dz = h2.z - h1.z;
                     const float dx = (h1.x + tx * dz) - h2.x;
                     const float dy = (h1.y + ty * dz) - h2.y;
                     const float sc = (dx * dx) + (dy * dy);
                     const unsigned long long key = ((unsigned long long)__float_as_uint(sc) << 32) |
                                                    __builtin_amdgcn_alignbit(id0, h2.qid, 16);
                     const bool better = in && key < bkey;
                     bkey = better ? key : bkey;
                     bpos = better ? (uint32_t)p : bpos;
                     if (KQ != 4) bp0 = better ? (uint32_t)pos0 : bp0;
                 });
            if (KQ == 4) bp0 = (uint32_t)pos0;
        }
        bpos |= bp0 << 16;
        group_min<KQ>(bkey, bpos, G);   // keys under the bound are unique
        const bool found = bkey != none && on;
        const unsigned long long em = __ballot(found && c == 0);
        if (em == 0ull) continue;
        // the table's slots are taken before the search and needed after it
        int slot = 0;
        if (lane == 0) slot = atomicAdd(&S.ctl[st.t & 1], __popcll(em));
        const uint32_t pos0 = bpos >> 16, pos2 = bpos & 0xFFFFu;
        unsigned long long bk = none_f;
        uint32_t pb = kNoPos;
        const int u = st.t + 1;
        if (more && st.n[5] > 0) {
            if (found && (KQ == 4 || c == 0)) {
                const Hit16 h2 = at(wc.h, pos2);
                const float d12 = h2.z - h1.z;
                const float tx = (h2.x - h1.x) / d12, ty = (h2.y - h1.y) / d12;
                follow_walk<2>(lds_window<CAP>(lo, u, st.n[5]), h2.x, h2.y, h2.z, tx, ty, st.Zn,
                            P.Wf, KQ == 4 ? c : 0, KQ == 4 ? 4 : 1, bk, pb);
            }
            if (KQ == 4) group_min<KQ>(bk, pb, G);
        }
        const float bsc = __uint_as_float((uint32_t)(bk >> 32));
        slot = uni(slot);
        if (found && (KQ == 4 || c == 0)) {
            const int l = slot + lane_rank(em) - (c > 0 ? 1 : 0);
            uint32_t *cl = Lay<CAP>::claim(lo);
            uint32_t *sd = Lay<CAP>::seeds(lo);
            uint16_t *sd16 = Lay<CAP>::seeds16(lo);
            const uint32_t kap = claim32(bsc, u);
            const uint32_t w0 = pos0 | ((uint32_t)p1 << 11) | (pos2 << 22), w1 = (pos2 >> 10) | (pb << 1),
                           w2 = __float_as_uint(bsc);
            const uint32_t a0 = (uint32_t)st.c[0] + pb, a1 = (uint32_t)st.c[2] + pos0, a2 = (uint32_t)(st.c[3] + p1),
                           a3 = (uint32_t)st.c[4] + pos2;
            const bool claims = pb != kNoPos && !gc;
            bool tie = false;
            if (KQ == 4) {
                // a lane of the quad for each claim and each word
                if (claims) tie = atomicMin(&cl[c == 0 ? a0 : c == 1 ? a1 : c == 2 ? a2 : a3], kap) == kap;
                if (c < 2) sd[c * CAP + l] = c == 0 ? w0 : w2;
                else if (c == 2) sd16[l] = (uint16_t)w1;
            } else {
                if (claims) {
                    const uint32_t o0 = atomicMin(&cl[a0], kap), o1 = atomicMin(&cl[a1], kap);
                    const uint32_t o2 = atomicMin(&cl[a2], kap), o3 = atomicMin(&cl[a3], kap);
                    tie = o0 == kap || o1 == kap || o2 == kap || o3 == kap;
                }
                sd[l] = w0;
                sd[CAP + l] = w2;
                sd16[l] = (uint16_t)w1;
            }
            if (tie) S.ctl[2] = 1;
        }
    }
    __builtin_amdgcn_s_setprio(0);
}

// hit i of a module, prefetched, and the word of the one before it
struct Fetch {
    Hit16 h;
    uint32_t qp;
};

// Every lane loads (an idle one the module's first entry; the entry behind
// the last module's is workspace memory too), so that nothing waits for the
// load before the hit is put into the ring.
__device__ __forceinline__ Fetch fetch_hit(const Hit16 *hs, int g, int n, int i)
{
    Fetch f;
    const Hit16 *s = hs + g;
    const uint32_t x = i < n ? (uint32_t)i : 0u;
    f.h = at(s, x);
    f.qp = at(s, x > 0u ? x - 1u : 0u).qid;
    return f;
}

// The n sorted hits of traversal index u into its ring slot, their ids to
// memory for the compaction, and the slot's coarse index: entry b is the
// first position whose bin is b or above, so a position owns the bins above
// its predecessor's up to its own, the last one also those above.
template <int B, int CAP>
__device__ __forceinline__ void ring_put(uint32_t lo, const Hit16 *hs, uint16_t *sid, int u, int g, int n, int i0,
                                         const Fetch &f)
{
    Hit16 *ring = Lay<CAP>::ring(lo, u & (kSlots - 1));
    uint16_t *tab = Lay<CAP>::tab(lo, u & (kSlots - 1));
    sid += g;
    const int sh = tab_shift(n);
    if (i0 >= n) return;
    Hit16 h = f.h;
    uint32_t qp = f.qp;
    asm volatile("" : "+v"(qp));   // keeps its use, and the wait for it, here
    for (int i = i0; i < n; i += B) {
        if (i != i0) {
            h = at(hs + g, (uint32_t)i);
            qp = at(hs + g, (uint32_t)(i - 1)).qid;
        }
        ring[i] = h;
        at(sid, (uint32_t)i) = id_of(h);
        const int own = (int)((h.qid & 0xFFFFu) >> sh);
#pragma unroll 1
        for (int b = i > 0 ? (int)((qp & 0xFFFFu) >> sh) + 1 : 0; b <= own; ++b) tab[b] = (uint16_t)i;
        if (i == n - 1) {
#pragma unroll 1
            for (int b = own + 1; b < (1 << (16 - sh)); ++b) tab[b] = (uint16_t)n;
        }
    }
}

// Takes the seeds of step t-1 into the free lanes.
template <int B, int CAP, int SETS>
__device__ __forceinline__ void take_seeds(uint32_t lo, const Step &st, Trk (&T)[SETS], const int (&base)[SETS], int nnew)
{
    const Hit16 *r1 = Lay<CAP>::ring(lo, (st.t - 2) & (kSlots - 1)), *r2 = Lay<CAP>::ring(lo, (st.t - 1) & (kSlots - 1));
#pragma unroll
    for (int s = 0; s < SETS; ++s) {
        const unsigned long long fm = __ballot(T[s].lst == 0u);
        const int l = base[s] + lane_rank(fm);
        if (T[s].lst == 0u && l < nnew) {
            const uint32_t a = Lay<CAP>::seeds(lo)[l], c = Lay<CAP>::seeds(lo)[CAP + l], b = Lay<CAP>::seeds16(lo)[l];
            const uint32_t pos1 = (a >> 11) & 0x7FFu, pos2 = (a >> 22) | ((b & 1u) << 10);
            const Hit16 h1 = at(r1, pos1), h2 = at(r2, pos2);
            T[s].xa = h1.x; T[s].ya = h1.y; T[s].za = h1.z;
            T[s].xb = h2.x; T[s].yb = h2.y; T[s].zb = h2.z;
            const uint32_t p0 = (uint32_t)st.g[1] + (a & 0x7FFu), p1 = (uint32_t)st.g[2] + pos1,
                           p2 = (uint32_t)st.g[3] + pos2;
            T[s].k0 = (h1.qid >> 16) | (p0 << 16);
            T[s].h12 = p1 | (p2 << 16);
            T[s].lst = p2 | (3u << 16) | ((uint32_t)(st.t - 1) << 24);
            T[s].pb = b >> 1;
            T[s].bsc = __uint_as_float(c);
        }
    }
}

// Seeding and following over all modules with the windows in LDS.  Leaves
// the final records (v.fin()) and their number in S.cnt[3], the flags by
// sorted position in LDS (and in memory with writeback), the previous hit of
// every appended hit in the links and the ids by sorted position in v.sid().
// gc: every stage is settled over the words in memory (a bare seed may outlive
// the claim slots).  Returns false when a step had more tracks than the lanes
// hold; the event is then run again from memory.
template <int B, int CAP, bool kCand>
__device__ __forceinline__ bool track_lds(const Ev &v0, Shared<B> &S, bool writeback, bool gc)
{
    constexpr int NW = B / 64, SETS = track_sets<B, CAP>();
    const int N = v0.N;
    const int lane = (int)(tid<B>() & 63), wv = uni((int)(tid<B>() >> 6));
    const int ri = (NW - 1 - wv) * 64 + lane;   // lanes counted from the last wave down
    uint32_t *own = Lay<CAP>::own(v0.lo);
    uint32_t *cl = Lay<CAP>::claim(v0.lo);
    const int nw = (N + 31) >> 5;
    const Hit16 *hs = v0.hs();
    uint16_t *link = v0.link(), *sid = v0.sid();
    Fin *fin = v0.fin();
    unsigned long long *claim = v0.claim();
    const uint32_t lo = v0.lo;
    const uint32_t *cand = kCand ? v0.keys() : nullptr;   // pendulum starts of a candidate pass

    const Prm P = fresh(kernel_params());
    Step st;
    int last_seed = 2;
    Trk T[SETS];
    {
    const sbt_params &PP = kernel_params();
    const int M = PP.n_modules;
    st.t = 2;
    st.g[0] = st.g[1] = st.n[0] = st.n[1] = 0;
#pragma unroll
    for (int i = 2; i < 7; ++i) {
        const int u = i - 2, k = u < M ? kmod(PP, u) : 0;
        st.g[i] = uni(S.mo[k]);
        st.n[i] = u < M ? uni(S.mo[k + 1] - S.mo[k]) : 0;
    }
    Fetch f0[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) f0[u] = fetch_hit(hs, st.g[u + 2], st.n[u + 2], ri);
    for (int i = tid<B>(); i < nw + 2; i += B) at(own, i) = 0u;
    for (int i = tid<B>(); i < kClaimSlots * CAP; i += B) cl[i] = 0xFFFFFFFFu;
    for (int i = tid<B>(); i < N; i += B) at(reinterpret_cast<uint32_t *>(link), (uint32_t)i) = 0xFFFFFFFFu;
    if (writeback)
        for (int i = tid<B>(); i < N; i += B) at(claim, (uint32_t)i) = kNoClaim;
    if (tid<B>() < 4) S.ctl[tid<B>()] = 0;
    if (tid<B>() < SBT_MAX_MODULES) {
        // the first step finds every slot free
        const int u = (int)tid<B>(), k = u < M ? kmod(PP, u) : 0, h = u / NW;
        const int w = h >= free_words<B, CAP>() ? 0 : 2 * h + 1 < SETS ? 64 | (64 << 16) : 64;
        S.mt[u] = make_int4(S.mo[k], S.mo[k + 1] - S.mo[k], __float_as_int(PP.module_z[k]), w);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (u < M) ring_put<B, CAP>(lo, hs, sid, u, st.g[u + 2], st.n[u + 2], ri, f0[u]);
    // the last traversal index whose seeding can make a seed: its modules
    // t-2, t-1 and t all hold hits (2 when no index can)
    {
        const unsigned long long hold = __ballot(lane < M && S.mo[kmod(PP, lane < M ? lane : 0) + 1] > S.mo[kmod(PP, lane < M ? lane : 0)]);
        const unsigned long long can = hold & (hold << 1) & (hold << 2);
        if (can) last_seed = 63 - __builtin_clzll(can);
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) st.c[i] = ((st.t + 1 + i) % 5) * CAP;   // slot of t - 4 + i
    st.Zc = PP.module_z[kmod(PP, 2)];
    st.Zn = M > 3 ? PP.module_z[kmod(PP, 3)] : 0.0f;
    st.Zx = M > 4 ? PP.module_z[kmod(PP, 4)] : 0.0f;
#pragma unroll
    for (int s = 0; s < SETS; ++s) T[s].lst = 0u;
    }
    ev_sync<B>();

    // base[s]: free slots of set s before this wave's (sets in order, waves
    // in order within a set); returns the number of free slots
    auto free_slots = [&](const int (&fsl)[(SETS + 1) / 2], int (&base)[SETS]) -> int {
        int total = 0;
#pragma unroll
        for (int h = 0; h < (SETS + 1) / 2; ++h) {
            const int x = fsl[h];
            const int inc = half_wave_incl_scan(x), ex = inc - x;
            const int mine = __builtin_amdgcn_readlane(ex, wv), all = __builtin_amdgcn_readlane(inc, 31);
            base[2 * h] = total + (mine & 0xFFFF);
            total += all & 0xFFFF;
            if (2 * h + 1 < SETS) {
                base[2 * h + 1 < SETS ? 2 * h + 1 : 0] = total + (mine >> 16);
                total += all >> 16;
            }
        }
        return total;
    };
    auto finish = [&](Trk &t, bool done) {
        const int r = wave_append(done, &S.ctl[3]);
        if (done) {
            Fin w;
            w.x = t.k0;
            w.y = t.h12;
            w.z = t.lst & 0xFFFFFFu;
            w.w = 0;
            at(fin, (uint32_t)r) = w;
            t.lst = 0u;
        }
    };
    Fetch f;
    bool ended = false, cleared = writeback;   // claims in memory: whether they have been cleared
    for (;;) {
        // ---- S(t)
        const bool more = st.t + 1 < P.M;
        f = fetch_hit(hs, st.g[6], st.n[6], ri);   // module t+2, put into the ring in R(t+1)
        if (st.n[2] > 0 && st.n[3] > 0 && st.n[4] > 0) {
            Free fr;
            static_assert(CAP <= 64 * 32, "the flag words of a module on half a wave");
            fr.a = free_word(own, st.g[2], st.n[2], lane);
            const unsigned long long fb = free_word(own, st.g[3], st.n[3], lane);
            const int pc = __popcll(fr.a) | (__popcll(fb) << 16);
            const int inc = half_wave_incl_scan(pc);
            const int tot = __builtin_amdgcn_readlane(inc, 31);
            const int ex = inc - pc;
            fr.ex = ex & 0xFFFF;
            fr.na = tot & 0xFFFF;
            fr.nb = tot >> 16;
            if (fr.na > 0 && fr.nb > 0) {
                // the lists of A's and Bm's unflagged positions, a word of
                // each per wave and round
                uint16_t *F = Lay<CAP>::freel(lo), *FM = Lay<CAP>::freem(lo);
                const int most = max(st.n[2], st.n[3]);
                for (int w = wv; 64 * w < most; w += NW) {
                    const unsigned long long ma = read_lane64(fr.a, w), mb = read_lane64(fb, w);
                    const int at0 = __builtin_amdgcn_readlane(ex, w);
                    if (__builtin_amdgcn_inverse_ballot_w64(ma))
                        at(F, (uint32_t)((at0 & 0xFFFF) + lane_rank(ma))) = (uint16_t)(64 * w + lane);
                    if (__builtin_amdgcn_inverse_ballot_w64(mb))
                        at(FM, (uint32_t)((at0 >> 16) + lane_rank(mb))) = (uint16_t)(64 * w + lane);
                }
                ev_lds_sync<B>();
                if (P.K == 4) seed_pass<B, CAP, 4, kCand>(P, lo, cand, st, S, fr, more, gc);
                else seed_pass<B, CAP, 0, kCand>(P, lo, cand, st, S, fr, more, gc);
            }
        }
        if (more) {
            const int u = st.t + 1;
            const LWin wn = lds_window<CAP>(lo, u, st.n[5]);
            const unsigned long long none_f = bound_key(P.Sf);
#pragma unroll
            for (int s = 0; s < SETS; ++s) {
                Trk &t = T[s];
                if (__ballot(t.lst != 0u) == 0ull) continue;
                t.pb = kNoPos;
                const int last_t = (int)(t.lst >> 24);
                const bool bare = ((t.lst >> 16) & 0xFFu) == 3u;
                const uint32_t p0 = t.k0 >> 16, p1 = t.h12 & 0xFFFFu, p2 = t.h12 >> 16;
                bool elig = t.lst != 0u && u - last_t <= P.misses + 1 && wn.n > 0;
                if (elig && bare) elig = is_free(own, p0) && is_free(own, p1) && is_free(own, p2);
                if (elig) {
                    const float dab = t.zb - t.za;
                    const float tx = (t.xb - t.xa) / dab, ty = (t.yb - t.ya) / dab;
                    unsigned long long bk = none_f;
                    follow_walk<walk_unroll(CAP)>(wn, t.xb, t.yb, t.zb, tx, ty, st.Zn, P.Wf, 0, 1, bk, t.pb);
                    t.bsc = __uint_as_float((uint32_t)(bk >> 32));
                    if (t.pb != kNoPos && !gc) {
                        // a kept bare seed was made at t-1: its hits are in t-3, t-2 and t-1
                        const uint32_t kap = claim32(t.bsc, u);
                        bool tie = atomicMin(&cl[(uint32_t)st.c[0] + t.pb], kap) == kap;
                        if (bare) {
                            const uint32_t o0 = atomicMin(&cl[st.c[1] + ((int)p0 - st.g[1])], kap);
                            const uint32_t o1 = atomicMin(&cl[st.c[2] + ((int)p1 - st.g[2])], kap);
                            const uint32_t o2 = atomicMin(&cl[st.c[3] + ((int)p2 - st.g[3])], kap);
                            tie = tie || o0 == kap || o1 == kap || o2 == kap;
                        }
                        if (tie) S.ctl[2] = 1;
                    }
                }
            }
        }
        ev_lds_sync<B>();
        // ---- on to t+1
        {
        const int M = P.M;
        st.t += 1;
        // everything the step's scalars come from, in one round of loads
        const int4 ctl = *reinterpret_cast<const int4 *>(S.ctl);
        const int4 nxt = S.mt[st.t + 2 < M ? st.t + 2 : 0];
        int fsl[(SETS + 1) / 2];
#pragma unroll
        for (int h = 0; h < (SETS + 1) / 2; ++h) fsl[h] = lane < NW ? free_at<B, CAP>(S, (st.t + 1) & 1, h, lane) : 0;
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            st.g[i] = st.g[i + 1];
            st.n[i] = st.n[i + 1];
        }
        {
            const int c0 = st.c[0];
#pragma unroll
            for (int i = 0; i < 4; ++i) st.c[i] = st.c[i + 1];
            st.c[4] = c0;
        }
        st.Zc = st.Zn;
        st.Zn = st.Zx;
        st.g[6] = uni(nxt.x);
        st.n[6] = st.t + 2 < M ? uni(nxt.y) : 0;
        st.Zx = __int_as_float(uni(nxt.z));
        const int t = st.t;
        int base[SETS];
        const int nnew = uni((t - 1) & 1 ? ctl.y : ctl.x);
        const int nfree = free_slots(fsl, base);
        const bool exact = gc || uni(ctl.z) != 0;
        if (nnew > nfree) return false;
        const bool end = t >= M;
        // with no forming track and no seed possible from here on, the
        // remaining steps change nothing
        ended = end || (nnew == 0 && nfree == SETS * B && t > last_seed);
        if (nnew > 0) take_seeds<B, CAP, SETS>(lo, st, T, base, nnew);
        if (ended) break;
        // ---- R(t)
        if (t + 1 < M) ring_put<B, CAP>(lo, hs, sid, t + 1, st.g[5], st.n[5], ri, f);
        if (exact) {
            // the claims of this stage over again as 64-bit words in memory
            if (!cleared)
                for (int i = tid<B>(); i < N; i += B) at(claim, (uint32_t)i) = kNoClaim;
            cleared = true;
            ev_sync<B>();
            if (tid<B>() == 0) S.ctl[2] = 0;
#pragma unroll
            for (int s = 0; s < SETS; ++s) {
                const Trk &k = T[s];
                if (k.lst == 0u || k.pb == kNoPos) continue;
                const unsigned long long kap = claim_key(k.bsc, (uint16_t)(k.k0 & 0xFFFFu), t);
                atomicMin(&at(claim, (uint32_t)st.g[4] + k.pb), kap);
                if (((k.lst >> 16) & 0xFFu) == 3u) {
                    atomicMin(&at(claim, k.k0 >> 16), kap);
                    atomicMin(&at(claim, k.h12 & 0xFFFFu), kap);
                    atomicMin(&at(claim, k.h12 >> 16), kap);
                }
            }
            ev_sync<B>();
        }
        Hit16 *rt = Lay<CAP>::ring(lo, t & (kSlots - 1));
        int nf[(SETS + 1) / 2 * 2] = {};
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
            Trk &k = T[s];
            const bool act = k.lst != 0u;
            if (__ballot(act) == 0ull) {
                nf[s] = 64;
                continue;
            }
            const int last_t0 = (int)(k.lst >> 24);
            const bool bare = ((k.lst >> 16) & 0xFFu) == 3u;
            const uint32_t p0 = k.k0 >> 16, p1 = k.h12 & 0xFFFFu, p2 = k.h12 >> 16;
            bool win = false;
            if (act && k.pb != kNoPos) {
                if (exact) {
                    const unsigned long long kap = claim_key(k.bsc, (uint16_t)(k.k0 & 0xFFFFu), t);
                    win = at(claim, (uint32_t)st.g[4] + k.pb) == kap;
                    if (bare) win = win && at(claim, p0) == kap && at(claim, p1) == kap && at(claim, p2) == kap;
                } else {
                    const uint32_t kap = claim32(k.bsc, t);
                    win = cl[(uint32_t)st.c[4] + k.pb] == kap;
                    if (bare) {
                        // made at t-1 (hits in t-3 .. t-1) or at t-2 (t-4 .. t-2)
                        const bool s1 = last_t0 == t - 1;
                        const int b0 = s1 ? st.c[1] - st.g[1] : st.c[0] - st.g[0];
                        const int b1 = s1 ? st.c[2] - st.g[2] : st.c[1] - st.g[1];
                        const int b2 = s1 ? st.c[3] - st.g[3] : st.c[2] - st.g[2];
                        const uint32_t o0 = cl[b0 + (int)p0], o1 = cl[b1 + (int)p1], o2 = cl[b2 + (int)p2];
                        win = win && o0 == kap && o1 == kap && o2 == kap;
                    }
                }
            }
            if (win) {
                const uint32_t p = (uint32_t)st.g[4] + k.pb;
                set_flag(own, p);
                if (bare) {
                    set_flag(own, p0);
                    set_flag(own, p1);
                    set_flag(own, p2);
                }
                at(link, 2u * p) = (uint16_t)(k.lst & 0xFFFFu);
                const Hit16 h = at(rt, k.pb);
                // a flagged hit loses its coordinate here, so that the seeding
                // walk over this module passes it by (nothing else reads it)
                at(rt, k.pb).x = __builtin_nanf("");
                k.xa = k.xb; k.ya = k.yb; k.za = k.zb;
                k.xb = h.x; k.yb = h.y; k.zb = h.z;
                k.lst = p | ((((k.lst >> 16) & 0xFFu) + 1u) << 16) | ((uint32_t)t << 24);
            }
            const bool done = k.lst != 0u && t - (int)(k.lst >> 24) >= P.misses + 1;
            if (__ballot(done) != 0ull) finish(k, done);
            nf[s] = __popcll(__ballot(k.lst == 0u));
        }
        if (lane == 0) {
#pragma unroll
            for (int h = 0; h < (SETS + 1) / 2; ++h) free_at<B, CAP>(S, t & 1, h, wv) = nf[2 * h] | (nf[2 * h + 1] << 16);
            if (wv == 0) S.ctl[t & 1] = 0;
        }
        ev_lds_sync<B>();
        }
    }
#pragma unroll
    for (int s = 0; s < SETS; ++s)
        if (__ballot(T[s].lst != 0u) != 0ull) finish(T[s], T[s].lst != 0u);
    if (writeback)
        for (int i = tid<B>(); i < nw; i += B) at(v0.own(), i) = at(own, i);
    ev_sync<B>();
    if (tid<B>() == 0) S.cnt[3] = S.ctl[3];
    ev_sync<B>();
    return true;
}

// ================================================================ memory form
// Best third hit for one doublet: the key orders like the comparison
// (found, scatter, id0, id2) -- scatter bits << 32 | id0 << 16 | id2, ~0 when
// nothing was found (scatters are >= +0, so their bits order like the
// values); pos holds the window positions pos0 | pos2 << 16.
__device__ __forceinline__ void seed_doublet(const Win &wa, const Win &wc, const uint32_t *own, int pos0, float x1,
                                             float y1, float z1, float Zc, float Ss, uint16_t Ws, uint16_t span,
                                             unsigned long long &bkey, uint32_t &bpos)
{
    const Hit16 h0 = at(wa.h, pos0);
    const uint32_t id0 = id_of(h0);
    const float d01 = z1 - h0.z;
    const float tx = (x1 - h0.x) / d01;
    const float ty = (y1 - h0.y) / d01;
    const float dzc = Zc - z1;
    const uint16_t qe = phi16(x1 + tx * dzc, y1 + ty * dzc);
    const int nc = wc.n;
    if (nc == 0) return;
    const uint16_t lo = (uint16_t)(qe - Ws);
    int pc = win_lower_bound(wc, lo);
    if (pc == nc) pc = 0;
    Hit16 h2n = at(wc.h, pc);
    for (int jj = 0; jj < nc; ++jj) {
        const Hit16 h2 = h2n;
        const int pn = pc + 1 == nc ? 0 : pc + 1;
        h2n = at(wc.h, pn);   // the next position, loaded while this one is scored
        if ((uint16_t)(q_of(h2) - lo) > span) break;
        const uint32_t id2 = id_of(h2);
        const float dz = h2.z - z1;
        const float dx = (x1 + tx * dz) - h2.x;
        const float dy = (y1 + ty * dz) - h2.y;
        const float sc = (dx * dx) + (dy * dy);
        const unsigned long long k = ((unsigned long long)__float_as_uint(sc) << 32) | (id0 << 16) | id2;
        const bool better = is_free(own, id2) && (sc < Ss) && (k < bkey);
        bkey = better ? k : bkey;
        bpos = better ? ((uint32_t)pos0 | ((uint32_t)pc << 16)) : bpos;
        pc = pn;
    }
}

// Following search of one forming track into traversal index u (Section 3,
// "track following"): the last two hits extrapolated to the module's
// nominal z, the best unflagged hit of the inclusive phi window by
// (scatter, id) under the threshold, and claims on that hit (and on the
// three seed hits of a bare seed) keyed (scatter, key) for stage u.  Returns
// the best hit's id | window position << 16, or ~0.
__device__ __forceinline__ uint32_t follow_item(const Prm &P, const Win &wc, float Zc, const uint32_t *own,
                                                unsigned long long *claim, const Rec &R, int u, float &bsc_out)
{
    const float Sf = P.Sf;
    const uint16_t Wf = (uint16_t)P.Wf;
    const uint16_t span = (uint16_t)(2 * P.Wf);
    const int nc = wc.n;
    uint16_t best = kNone;
    int bpos = 0;
    float bsc = 0.0f;
    bool elig = (u - (int)R.last_t) <= P.misses + 1;
    if (elig && R.len == 3) elig = is_free(own, R.h0) && is_free(own, R.h1) && is_free(own, R.h2);
    if (elig && nc > 0) {
        const float dzc = Zc - R.zb;
        const uint16_t qe = phi16(R.xb + R.tx * dzc, R.yb + R.ty * dzc);
        const uint16_t lo = (uint16_t)(qe - Wf);
        int pc = win_lower_bound(wc, lo);
        if (pc == nc) pc = 0;
        // No hit of module u is flagged yet: flags are set only when a
        // module is resolved, and u is resolved after this search.  The
        // flag test of the method is therefore always passed here.
        // (scatter, id) packed so that one comparison orders both
        unsigned long long bk = ~0ull;
        Hit16 hn = at(wc.h, pc);
        for (int j = 0; j < nc; ++j) {
            const Hit16 h = hn;
            const int pn = pc + 1 == nc ? 0 : pc + 1;
            hn = at(wc.h, pn);   // the next position, loaded while this one is scored
            if ((uint16_t)(q_of(h) - lo) > span) break;
            const float dz = h.z - R.zb;
            const float dx = (R.xb + R.tx * dz) - h.x;
            const float dy = (R.yb + R.ty * dz) - h.y;
            const float sc = (dx * dx) + (dy * dy);
            const unsigned long long k = ((unsigned long long)__float_as_uint(sc) << 32) | id_of(h);
            const bool better = (sc < Sf) && (k < bk);
            bk = better ? k : bk;
            bpos = better ? pc : bpos;
            pc = pn;
        }
        if (bk != ~0ull) {
            best = (uint16_t)(bk & 0xFFFFu);
            bsc = __uint_as_float((uint32_t)(bk >> 32));
        }
        if (best != kNone) {
            const unsigned long long kap = claim_key(bsc, R.key, u);
            atomicMin(&at(claim, best), kap);
            if (R.len == 3) {
                atomicMin(&at(claim, R.h0), kap);
                atomicMin(&at(claim, R.h1), kap);
                atomicMin(&at(claim, R.h2), kap);
            }
        }
    }
    bsc_out = bsc;
    return best == kNone ? 0xFFFFFFFFu : ((uint32_t)bpos << 16) | best;
}

// Seeding(t), t >= 2 (Section 3), fused with the following search into
// t+1.  With kCand the pendulum start of every middle hit is read from the
// table a separate candidate pass wrote into the workspace (the paper's
// "Fill candidates" kernel) instead of being searched here.  Seeding: modules
// A = kmod(t-2), Bm = kmod(t-1), C = kmod(t); work items are (unflagged middle
// hit, partner rank c) -- with K a power of two up to 16, the K doublets of a
// middle hit run on K adjacent lanes and their best triplets are reduced
// across the lanes, otherwise one lane handles all K.  A new seed's following
// search into t+1 runs on the lane that made it.  The tracks kept by the last
// resolution (active slots [0, n_keep)) search t+1 on waves of their own.
// Both read the flags as the resolution of t left them, which is the state
// the following of t+1 starts from.
template <int B, bool kCand>
__device__ __forceinline__ void stage_seed_follow(const sbt_params &PP, const Ev &v0, int t, Shared<B> &S, const uint32_t *own,
                                  uint16_t *nxt, int *n_nxt, int n_keep, bool follow_next)
{
    const Prm P = fresh(PP);
    const Ev v = fresh(v0);
    const Win wa = window<B>(P, S, v, t - 2);
    const Win wb = window<B>(P, S, v, t - 1);
    const Win wc = window<B>(P, S, v, t);
    Win wn = wc;
    float Zn = 0.0f;
    if (follow_next) {
        wn = window<B>(P, S, v, t + 1);
        Zn = PP.module_z[kmod(P, t + 1)];
    }
    const int na = wa.n, nbm = wb.n;
    const float Zc = PP.module_z[kmod(P, t)];
    const float Ss = P.Ss;
    const int K = P.K;
    const uint16_t Ws = (uint16_t)P.Ws;
    const uint16_t span = (uint16_t)(2 * P.Ws);

    // unflagged positions of the doublet module and of the middle module, ascending
    const int ga = uni(S.mo[kmod(P, t - 2)]), gb = uni(S.mo[kmod(P, t - 1)]);
    uint16_t *F = v.list(kListFreeL) + ga;
    uint16_t *FR = v.list(kListFRank) + ga;
    uint16_t *FM = v.list(kListFreeM) + gb;
    int nf = 0, nfm = 0;
    const int nmax = na > nbm ? na : nbm;
    int phase = 0;
    for (int base = 0; base < nmax; base += B, ++phase) {
        const int p = base + (int)tid<B>();
        const bool fa = p < na && is_free(own, win_id(wa, p));
        const bool fb = p < nbm && is_free(own, win_id(wb, p));
        int total;
        const int idx = block_count2<B>(fa, fb, S.scan, phase, &total);
        if (p < na) at(FR, p) = (uint16_t)(nf + (idx & 0xFFFF));
        if (fa) at(F, nf + (idx & 0xFFFF)) = (uint16_t)p;
        if (fb) at(FM, nfm + (idx >> 16)) = (uint16_t)p;
        nf += total & 0xFFFF;
        nfm += total >> 16;
    }
    ev_sync<B>();
    const int hd = na >> 1, hu = na - hd - 1;   // offsets visited: [-hd, hu]
    const int G = (K == 1 || K == 2 || K == 4 || K == 8 || K == 16) ? K : 1;
    const int per_lane = G == 1 ? K : 1;
    const int seed_items = (nf > 0 && nfm > 0) ? nfm * G : 0;
    const int seed_pad = (seed_items + 63) & ~63;      // seeding and following never share a wave
    const int follow_items = follow_next ? n_keep : 0;
    const int total = seed_pad + follow_items;

    for (int base = 0; base < total; base += B) {
        const int g = base + (int)tid<B>();
        const int g_wave = uni(base + ((int)tid<B>() & ~63));
        if (g_wave >= seed_pad) {
            const int a = g - seed_pad;
            if (a < follow_items) {
                const int r = at(nxt, a);
                const Rec R = at(v.rec(), r);
                float bsc;
                const uint32_t pb = follow_item(P, wn, Zn, own, v.claim(), R, t + 1, bsc);
                RecAux &x = at(v.aux(), r);
                x.best = pb;
                x.bsc = bsc;
            }
            continue;
        }
        // the seeding waves carry the longest dependency chain of the step
        __builtin_amdgcn_s_setprio(2);
        const int i = g / G, c = g - i * G;
        unsigned long long bkey = ~0ull;
        uint32_t bpos = 0;
        Hit16 h1;
        h1.x = h1.y = h1.z = 0.0f;
        h1.qid = 0;
        if (g < seed_items) {
            const int p1 = at(FM, i);
            h1 = at(wb.h, p1);
            int s0;
            if (kCand) {
                s0 = (int)at(v.keys(), (uint32_t)(gb + p1));
            } else {
                s0 = win_lower_bound(wa, q_of(h1));
                if (s0 == na) s0 = 0;
            }
            const int j = at(FR, s0);   // first unflagged position >= s0, as an index into F
            if (G == 4) {
                const int pos0 = pendulum_quad(F, nf, j, s0, na, hu, hd, c);
                if (pos0 >= 0) seed_doublet(wa, wc, own, pos0, h1.x, h1.y, h1.z, Zc, Ss, Ws, span, bkey, bpos);
            } else {
                for (int cc = 0; cc < per_lane; ++cc) {
                    const int pos0 = pendulum_pick(F, nf, j, s0, na, hu, hd, c + cc);
                    if (pos0 < 0) break;
                    seed_doublet(wa, wc, own, pos0, h1.x, h1.y, h1.z, Zc, Ss, Ws, span, bkey, bpos);
                }
            }
        }
        // minimum over the G lanes of a middle hit (keys are unique or ~0)
        for (int m = 1; m < G; m <<= 1) {
            const uint32_t olo = (uint32_t)lane_xor((int)(uint32_t)bkey, m);
            const uint32_t ohi = (uint32_t)lane_xor((int)(uint32_t)(bkey >> 32), m);
            const uint32_t opos = (uint32_t)lane_xor((int)bpos, m);
            const unsigned long long o = ((unsigned long long)ohi << 32) | olo;
            if (o < bkey) {
                bkey = o;
                bpos = opos;
            }
        }
        const bool emit = bkey != ~0ull && c == 0 && g < seed_items;
        int r, l;
        wave_append2(emit, &S.cnt[0], emit, n_nxt, r, l);
        if (emit) {
            const int pos0 = (int)(bpos & 0xFFFFu), pos2 = (int)(bpos >> 16);
            const Hit16 h0 = at(wa.h, pos0);
            const Hit16 h2 = at(wc.h, pos2);
            const float x1 = h1.x, y1 = h1.y, z1 = h1.z;
            Rec R;
            const float d12 = h2.z - z1;
            R.xb = h2.x; R.yb = h2.y; R.zb = h2.z;
            R.tx = (h2.x - x1) / d12;
            R.ty = (h2.y - y1) / d12;
            R.key = id_of(h1); R.h0 = id_of(h0); R.h1 = id_of(h1); R.h2 = id_of(h2); R.last = id_of(h2);
            R.len = 3; R.last_t = (uint8_t)t;
            at(v.rec(), r) = R;
            at(v.aux(), r).chi2 = seed_chi2(h0, h1, h2);
            at(nxt, l) = (uint16_t)r;
            if (follow_next) {
                float bsc;
                const uint32_t pb = follow_item(P, wn, Zn, own, v.claim(), R, t + 1, bsc);
                RecAux &x = at(v.aux(), r);
                x.best = pb;
                x.bsc = bsc;
            }
        }
        __builtin_amdgcn_s_setprio(0);
    }
}

// A track wins iff its key is the minimum on every hit it claimed; winners
// append their best hit and flag their claim set.  Tracks that have now missed
// more than max_consecutive_misses modules in a row become final; the others
// stay active for the next module.
template <int B>
__device__ __forceinline__ void stage_follow_resolve(const sbt_params &PP, const Ev &v0, int t, Shared<B> &S, uint32_t *own,
                                     const uint16_t *act, int n_act, uint16_t *nxt, int *n_nxt)
{
    const Prm P = fresh(PP);
    const Ev v = fresh(v0);
    const Win wc = window<B>(P, S, v, t);
    const unsigned long long *__restrict__ claim = v.claim();
    uint16_t *fin = v.list(kListFin);
    for (int base = 0; base < n_act; base += B) {
        const int a = base + (int)tid<B>();
        bool done = false, keep = false;
        int r = 0;
        if (a < n_act) {
            r = at(act, a);
            const RecAux &x = at(v.aux(), r);
            const uint32_t pb = x.best;
            const float bsc = x.bsc;
            Rec R = at(v.rec(), r);
            const uint16_t best = (uint16_t)(pb & 0xFFFF);
            bool win = false;
            if (pb != 0xFFFFFFFFu) {
                const unsigned long long kap = claim_key(bsc, R.key, t);
                win = at(claim, best) == kap;
                if (R.len == 3)
                    win = win && at(claim, R.h0) == kap && at(claim, R.h1) == kap && at(claim, R.h2) == kap;
            }
            int last_t = R.last_t;
            if (win) {
                const int bpos = (int)(pb >> 16);
                set_flag(own, best);
                if (R.len == 3) {
                    set_flag(own, R.h0);
                    set_flag(own, R.h1);
                    set_flag(own, R.h2);
                }
                at(v.link(), 2u * best) = R.last;
                const Hit16 hn = at(wc.h, bpos);
                const float dab = hn.z - R.zb;
                R.tx = (hn.x - R.xb) / dab;
                R.ty = (hn.y - R.yb) / dab;
                R.xb = hn.x; R.yb = hn.y; R.zb = hn.z;
                R.last = best;
                R.len = (uint8_t)(R.len + 1);
                R.last_t = (uint8_t)t;
                at(v.rec(), r) = R;
                last_t = t;
            }
            done = (t - last_t) >= P.misses + 1;
            keep = !done;
        }
        int f, l;
        wave_append2(done, &S.cnt[3], keep, n_nxt, f, l);
        if (done) at(fin, f) = (uint16_t)r;
        if (keep) at(nxt, l) = (uint16_t)r;
    }
}

// Seeding and following over all modules from memory.  Leaves the final
// record list in the final list and its length in S.cnt[3].
template <int B, bool kCand>
__device__ __forceinline__ void track_mem(const sbt_params &PP, const Ev &v, Shared<B> &S)
{
    const Prm P = fresh(PP);
    const int M = P.M, N = v.N;
    uint32_t *own = v.own();
    const int nw = (N + 31) >> 5;
    for (int i = tid<B>(); i < nw; i += B) at(own, i) = 0u;
    for (int i = tid<B>(); i < N; i += B) {
        at(v.claim(), i) = kNoClaim;
        at(v.link(), 2u * i + 1u) = kNone;
    }
    if (tid<B>() == 0) {
        S.cnt[0] = 0; S.cnt[1] = 0; S.cnt[2] = 0; S.cnt[3] = 0;
    }
    ev_sync<B>();
    uint16_t *l0 = v.list(kListAct0);
    uint16_t *l1 = v.list(kListAct1);
    // the last traversal index whose seeding can make a seed: its modules
    // t-2, t-1 and t all hold hits (2 when no index can)
    int last_seed = 2;
    for (int u = M - 1; u > 2; --u) {
        const int k0 = kmod(P, u), k1 = kmod(P, u - 1), k2 = kmod(P, u - 2);
        if (S.mo[k0 + 1] > S.mo[k0] && S.mo[k1 + 1] > S.mo[k1] && S.mo[k2 + 1] > S.mo[k2]) {
            last_seed = u;
            break;
        }
    }
    last_seed = uni(last_seed);
    int par = 0;
    stage_seed_follow<B, kCand>(PP, v, 2, S, own, l0, &S.cnt[1], 0, M > 3);
    ev_sync<B>();
    for (int t = 3; t < M; ++t) {
        // act (n_act tracks) holds every forming track with its search into
        // t done: resolve t keeping the survivors in nxt, then seed t and
        // search t+1
        const int n_act = uni(S.cnt[1 + par]);
        // with no forming track and no seed possible from here on, the
        // remaining steps change nothing
        if (n_act == 0 && t > last_seed) break;
        uint16_t *act = par ? l1 : l0;
        uint16_t *nxt = par ? l0 : l1;
        const bool more = t + 1 < M;
        stage_follow_resolve<B>(PP, v, t, S, own, act, n_act, nxt, &S.cnt[1 + (par ^ 1)]);
        ev_sync<B>();
        const int n_keep = uni(S.cnt[1 + (par ^ 1)]);
        if (tid<B>() == 0) S.cnt[1 + par] = 0;   // act becomes the next step's nxt
        stage_seed_follow<B, kCand>(PP, v, t, S, own, nxt, &S.cnt[1 + (par ^ 1)], n_keep, more);
        ev_sync<B>();
        par ^= 1;
    }
    const int n_act = uni(S.cnt[1 + par]);
    const int nf = uni(S.cnt[3]);
    const uint16_t *act = par ? l1 : l0;
    uint16_t *fin = v.list(kListFin);
    for (int a = tid<B>(); a < n_act; a += B) at(fin, nf + a) = at(act, a);
    ev_sync<B>();
    if (tid<B>() == 0) S.cnt[3] = nf + n_act;
    ev_sync<B>();
}

// whether an event fits the LDS form of the tracking stages
template <int B, int CAP>
__device__ __forceinline__ bool event_fits_lds(const Shared<B> &S, int N, int own_cap)
{
    return CAP > 0 && uni(S.maxmod) <= CAP && N <= own_cap;
}

// Runs the tracking stages; returns true when they ran in the LDS form
// (flags in LDS, hits named by sorted position), false for the memory form.
template <int B, int CAP, bool kCand = false>
__device__ __forceinline__ bool stage_track(const sbt_params &P, const Ev &v, Shared<B> &S, int own_cap, bool writeback)
{
    if constexpr (CAP > 0) {
        if (event_fits_lds<B, CAP>(S, v.N, own_cap)) {
            // a bare seed that may miss two modules outlives the claim slots
            const bool gc = P.max_consecutive_misses > 1;
            if (track_lds<B, CAP, kCand>(fresh(v), S, writeback, gc)) return true;
            ev_sync<B>();   // every wave has read what made it return
        }
    }
    track_mem<B, kCand>(P, v, S);
    return false;
}

// ---------------------------------------------------------------- candidate pass
// The paper's separate "Fill candidates" step, as an ablation of the fused
// search: for every hit of every module after the first in traversal order,
// the first position of the preceding module (in traversal order: the
// doublet module when this hit is a middle hit) whose phi16 is >= the hit's,
// 0 when there is none -- the pendulum start, which does not depend on the
// flags.  Written by sorted position into the keys array (free after the
// sort) for the seeding stage to read.
template <int B>
__device__ void stage_fill_candidates(const sbt_params &PP, const Ev &v0, const Shared<B> &S)
{
    const Ev v = fresh(v0);
    const Prm P = fresh(PP);
    for (int u = 1; u < P.M; ++u) {
        const int k = kmod(P, u), ka = kmod(P, u - 1);
        const int g0 = S.mo[k], n = S.mo[k + 1] - g0;
        Win wa;
        wa.h = v.hs() + S.mo[ka];
        wa.n = S.mo[ka + 1] - S.mo[ka];
        for (int i = tid<B>(); i < n; i += B) {
            int s0 = wa.n > 0 ? win_lower_bound(wa, q_of(at(v.hs(), (uint32_t)(g0 + i)))) : 0;
            if (s0 == wa.n) s0 = 0;
            at(v.keys(), (uint32_t)(g0 + i)) = (uint32_t)s0;
        }
    }
}

// ---------------------------------------------------------------- tracklet filter
// Tracks of >= 4 hits are accepted; a three-hit track is a candidate when its
// fit chi2 is under the threshold and none of its hits is flagged; candidates
// sharing hits keep the one with the minimum (chi2, key).
template <int B>
__device__ __forceinline__ void stage_filter(const sbt_params &PP, const Ev &v0, int n_fin, const uint32_t *own)
{
    const Ev v = fresh(v0);
    const float X = fresh(PP).X;
    unsigned long long *__restrict__ claim = v.claim();
    const uint16_t *fin = v.list(kListFin);
    for (int a = tid<B>(); a < n_fin; a += B) {
        const int r = at(fin, a);
        const Rec R = at(v.rec(), r);
        uint32_t fl = 0;
        if (R.len >= 4) {
            fl = kFlagAccepted;
        } else {
            const float c2 = at(v.aux(), r).chi2;
            if (c2 < X && is_free(own, R.h0) && is_free(own, R.h1) && is_free(own, R.h2)) {
                const unsigned long long kap = claim_key(c2, R.key, kFilterStage);
                atomicMin(&at(claim, R.h0), kap);
                atomicMin(&at(claim, R.h1), kap);
                atomicMin(&at(claim, R.h2), kap);
                fl = kFlagCandidate;
            }
        }
        at(v.aux(), r).flag = fl;
    }
    ev_sync<B>();
    for (int a = tid<B>(); a < n_fin; a += B) {
        const int r = at(fin, a);
        const RecAux x = at(v.aux(), r);
        uint32_t fl = x.flag;
        const Rec R = at(v.rec(), r);
        if (fl == kFlagCandidate) {
            const unsigned long long kap = claim_key(x.chi2, R.key, kFilterStage);
            fl = (at(claim, R.h0) == kap && at(claim, R.h1) == kap && at(claim, R.h2) == kap) ? kFlagAccepted : 0;
        }
        if (fl == kFlagAccepted) at(v.link(), 2u * R.key + 1u) = (uint16_t)r;
    }
    ev_sync<B>();
}

// The same for the LDS form's records.  claim: one word per sorted position,
// all ~0.
template <int B, class Claim>
__device__ __forceinline__ void filter_records(const Ev &v, float X, int n_fin, const uint32_t *own, Claim claim)
{
    for (int a = tid<B>(); a < n_fin; a += B) {
        const Fin w = at(v.fin(), (uint32_t)a);
        uint32_t fl = kFlagAccepted;
        if ((w.z >> 16) < 4u) {
            const uint32_t p0 = w.x >> 16, p1 = w.y & 0xFFFFu, p2 = w.y >> 16;
            const float c2 = seed_chi2(at(v.hs(), p0), at(v.hs(), p1), at(v.hs(), p2));
            fl = 0;
            if (c2 < X && is_free(own, p0) && is_free(own, p1) && is_free(own, p2)) {
                const unsigned long long kap = claim_key(c2, (uint16_t)(w.x & 0xFFFFu), kFilterStage);
                atomicMin(claim + p0, kap);
                atomicMin(claim + p1, kap);
                atomicMin(claim + p2, kap);
                fl = kFlagCandidate;
                at(v.aux(), (uint32_t)a).chi2 = c2;
            }
        }
        if (fl == kFlagAccepted) at(v.link(), 2u * (w.x & 0xFFFFu) + 1u) = (uint16_t)a;
        at(v.aux(), (uint32_t)a).flag = fl;
    }
    ev_sync<B>();
    for (int a = tid<B>(); a < n_fin; a += B) {
        const RecAux x = at(v.aux(), (uint32_t)a);
        if (x.flag != kFlagCandidate) continue;
        const Fin w = at(v.fin(), (uint32_t)a);
        const uint32_t p0 = w.x >> 16, p1 = w.y & 0xFFFFu, p2 = w.y >> 16;
        const unsigned long long kap = claim_key(x.chi2, (uint16_t)(w.x & 0xFFFFu), kFilterStage);
        if (claim[p0] == kap && claim[p1] == kap && claim[p2] == kap) at(v.link(), 2u * (w.x & 0xFFFFu) + 1u) = (uint16_t)a;
    }
    ev_sync<B>();
}

// own in LDS at byte offset own_off of the event's region, where the claims
// fit in front of it; claims in memory otherwise
template <int B>
__device__ __forceinline__ void stage_filter_lds(const sbt_params &PP, const Ev &v0, int n_fin, uint32_t own_off)
{
    const Ev v = fresh(v0);
    const float X = fresh(PP).X;
    const uint32_t *own = reinterpret_cast<const uint32_t *>(g_lds + v.lo + own_off);
    if (8u * (uint32_t)v.N <= own_off) {
        unsigned long long *claim = reinterpret_cast<unsigned long long *>(g_lds + v.lo);
        for (int i = tid<B>(); i < v.N; i += B) claim[i] = kNoClaim;
        ev_lds_sync<B>();
        filter_records<B>(v, X, n_fin, own, claim);
    } else {
        unsigned long long *claim = v.claim();
        for (int i = tid<B>(); i < v.N; i += B) at(claim, (uint32_t)i) = kNoClaim;
        ev_sync<B>();
        filter_records<B>(v, X, n_fin, own, claim);
    }
}

// own and claims in memory (the plain form's kernels; claims already ~0)
template <int B>
__device__ void stage_filter_pos(const sbt_params &PP, const Ev &v0, int n_fin)
{
    const Ev v = fresh(v0);
    filter_records<B>(v, fresh(PP).X, n_fin, v.own(), v.claim());
}

// ---------------------------------------------------------------- per-event compaction
// The accepted tracks in key order (the id of the seed's middle hit), each as
// its three seed hits followed by the hits appended to it in traversal order:
// per-event track offsets and hit ids into the staging arrays, counts into
// the event's counters.
constexpr int kCompactBatch = 8;   // key rounds whose link loads are in flight together

// An accepted track's record: the seed's hits, the last hit and the number of
// hits, by sorted position (kPos, the LDS tracking form's) or by id.
struct Acc {
    uint32_t h0, h1, h2, last, len;
};

template <bool kPos>
__device__ __forceinline__ Acc accepted(const Ev &v, uint32_t r)
{
    Acc a;
    if (kPos) {
        const Fin w = at(v.fin(), r);
        a.h0 = w.x >> 16;
        a.h1 = w.y & 0xFFFFu;
        a.h2 = w.y >> 16;
        a.last = w.z & 0xFFFFu;
        a.len = w.z >> 16;
    } else {
        const Rec R = at(v.rec(), r);
        a.h0 = R.h0;
        a.h1 = R.h1;
        a.h2 = R.h2;
        a.last = R.last;
        a.len = R.len;
    }
    return a;
}

// How the compaction of an event of N hits runs in lds_bytes of LDS: kWhole
// holds the previous-hit links (2 B per hit), with pos the ids by sorted
// position (2 B per hit), and the record of each accepted track in key order
// (2 B per track; tracks are disjoint with at least three hits, so at most
// N / 3); kIdsInMemory leaves the ids where they are, each read once beside
// the walk of the links (200 events of 16,120 hits in the plain form: 371 us,
// 685 with everything in memory; of 11,440 hits on 512 lanes with 480-hit
// slots 259 and 401; of 6,500 on 256 lanes with 256-hit slots 216 and 367).
enum class Compact { kMemory, kIdsInMemory, kWhole };
__host__ __device__ constexpr Compact compact_form(int N, int lds_bytes, bool pos)
{
    const int row = (int)a16(2u * (uint32_t)N), tracks = 2 * (N / 3 + 1);
    if ((pos ? 2 : 1) * row + tracks <= lds_bytes) return Compact::kWhole;
    return pos && row + tracks <= lds_bytes ? Compact::kIdsInMemory : Compact::kMemory;
}

// LDS form (kIds: the ids too).  Pass 1 takes the keys in rounds of B (key = round * B + lane,
// loads coalesced, kCompactBatch rounds in flight), copies each previous-hit
// link to LDS and ranks the keys that own a record with a ballot count over
// the workgroup, which lists the records in key order.  Pass 2 gives each
// listed track a lane: an exclusive scan of the lengths places its hits, and
// the lane writes them, walking the links in LDS.
template <int B, bool kPos, bool kIds>
__device__ __forceinline__ void compact_lds(const Ev &v, int *s_scan, int lds_bytes)
{
    const int N = v.N;
    const uint32_t row = a16(2u * (uint32_t)N);
    uint16_t *lprev = reinterpret_cast<uint16_t *>(g_lds + v.lo);
    uint16_t *lid = reinterpret_cast<uint16_t *>(g_lds + v.lo + row);   // kIds
    uint16_t *lrec = reinterpret_cast<uint16_t *>(g_lds + v.lo + (kIds ? 2 : 1) * row);
    const int rec_cap = (lds_bytes - (kIds ? 2 : 1) * (int)row) / 2;
    const uint32_t *link = reinterpret_cast<const uint32_t *>(v.link());   // prev | record << 16
    const int rounds = (N + B - 1) / B;
    auto id = [&](uint32_t p) -> uint16_t { return kIds ? lid[p] : kPos ? at(v.sid(), p) : (uint16_t)p; };
    bool bad = false;
    int nt = 0;
    for (int j0 = 0; j0 < rounds; j0 += kCompactBatch) {
        uint32_t w[kCompactBatch];
        uint16_t d[kCompactBatch];
#pragma unroll
        for (int u = 0; u < kCompactBatch; ++u) {
            const int k = (j0 + u) * B + (int)tid<B>();
            w[u] = k < N ? at(link, (uint32_t)k) : ((uint32_t)kNone << 16);
            if (kIds) d[u] = k < N ? at(v.sid(), (uint32_t)k) : (uint16_t)0;
        }
#pragma unroll
        for (int u = 0; u < kCompactBatch; ++u) {
            if (j0 + u >= rounds) break;
            const int k = (j0 + u) * B + (int)tid<B>();
            const uint16_t r = (uint16_t)(w[u] >> 16);
            if (k < N) {
                lprev[k] = (uint16_t)(w[u] & 0xFFFFu);
                if (kIds) lid[k] = d[u];
            }
            int tot;
            const int pos = nt + (block_count2<B>(r != kNone, false, s_scan, j0 + u, &tot) & 0xFFFF);
            if (r != kNone) {
                if (pos < rec_cap) lrec[pos] = r;
                else bad = true;
            }
            nt += tot & 0xFFFF;
        }
    }
    ev_sync<B>();   // links, ids and the record list visible
    if (nt > rec_cap) nt = 0;
    int nh = 0;
    for (int t0 = 0; t0 < nt; t0 += B) {
        const int t = t0 + (int)tid<B>();
        Acc R;
        R.len = 0;
        if (t < nt) R = accepted<kPos>(v, lrec[t]);
        const int len = (int)R.len;
        int tot;
        const int hi = nh + block_excl_scan<B>(len, s_scan, t0 / B, &tot);
        nh += tot;
        if (t < nt) {
            // tracks are disjoint, so hi + len <= N; the checks below only
            // keep a broken invariant from turning into a stray access
            if (hi + len > N) {
                bad = true;
            } else {
                at(v.st_toff(), t) = hi;
                uint16_t *out = v.st_hits() + hi;
                uint32_t p = R.last;
                for (int j = len - 1; j >= 3; --j) {
                    if (p >= (uint32_t)N) { bad = true; break; }
                    out[j] = id(p);
                    p = lprev[p];
                }
                out[2] = id(R.h2);
                out[1] = id(R.h1);
                out[0] = id(R.h0);
            }
        }
    }
    if (bad) v.info().st = (int)SBT_EV_INTERNAL;
    if (tid<B>() == 0) {
        v.info().nt = nh <= N ? nt : 0;
        v.info().nh = nh <= N ? nh : 0;
    }
}

// Memory form (events whose links do not fit, and the plain kernel): each
// lane owns a contiguous range of keys; it counts their tracks and hits, one
// scan of each over the workgroup, then it writes them in key order.
template <int B, bool kPos>
__device__ __forceinline__ void compact_mem(const Ev &v, int *s_scan)
{
    const int N = v.N;
    const int per = (N + B - 1) / B;
    const int k0 = min(N, (int)tid<B>() * per), k1 = min(N, k0 + per);
    int nt = 0, nh = 0;
    for (int k = k0; k < k1; ++k) {
        const uint16_t r = at(v.link(), 2u * k + 1u);
        if (r != kNone) {
            ++nt;
            nh += (int)accepted<kPos>(v, r).len;
        }
    }
    int tt, th;
    int ti = block_excl_scan<B>(nt, s_scan, 0, &tt);
    int hi = block_excl_scan<B>(nh, s_scan, 1, &th);
    bool bad = th > N;
    for (int k = k0; k < k1 && !bad; ++k) {
        const uint16_t r = at(v.link(), 2u * k + 1u);
        if (r == kNone) continue;
        const Acc R = accepted<kPos>(v, r);
        const int len = (int)R.len;
        if (hi + len > N) {
            bad = true;
            break;
        }
        at(v.st_toff(), ti) = hi;
        uint16_t *out = v.st_hits() + hi;
        uint32_t p = R.last;
        for (int j = len - 1; j >= 3; --j) {
            if (p >= (uint32_t)N) { bad = true; break; }
            out[j] = kPos ? at(v.sid(), p) : (uint16_t)p;
            p = at(v.link(), 2u * p);
        }
        out[2] = kPos ? at(v.sid(), R.h2) : (uint16_t)R.h2;
        out[1] = kPos ? at(v.sid(), R.h1) : (uint16_t)R.h1;
        out[0] = kPos ? at(v.sid(), R.h0) : (uint16_t)R.h0;
        ++ti;
        hi += len;
    }
    if (bad) v.info().st = (int)SBT_EV_INTERNAL;
    if (tid<B>() == 0) {
        v.info().nt = th <= N ? tt : 0;
        v.info().nh = th <= N ? th : 0;
    }
}

// lds_bytes: LDS free for the compaction (0: none).  kApart: kIdsInMemory is
// compiled in; its condition is hidden from the optimiser, which otherwise
// keeps parts of it live through the tracking stages (one event of 4,000 hits
// 2 % slower).
template <int B, bool kPos, bool kApart = kPos>
__device__ __forceinline__ void stage_compact(const Ev &v0, int *s_scan, int lds_bytes)
{
    const Ev v = fresh(v0);
    const Compact want = compact_form(v.N, lds_bytes, kPos);
    const Compact form = kApart ? (Compact)opq((int)want) : want;
    if (form == Compact::kWhole) compact_lds<B, kPos, kPos>(v, s_scan, lds_bytes);
    else if (kApart && form == Compact::kIdsInMemory) compact_lds<B, kPos, false>(v, s_scan, lds_bytes);
    else compact_mem<B, kPos>(v, s_scan);
}

}  // namespace sbt
