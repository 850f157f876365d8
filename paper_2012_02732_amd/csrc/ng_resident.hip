// The device-resident replay kernel. Compiled once per build of the kernel (NG_RESIDENT_BUILD: lean, full, train), each an
// object of its own, so that the three compile side by side.
#include "ng_kernels.hip"

#ifndef NG_RESIDENT_BUILD
#error "compile with -DNG_RESIDENT_BUILD=0, 1 or 2"
#endif

namespace ng {
namespace {

// ------------------------------------------------------------------------------------
// Device-resident replay. The recorded schedule (Section 4.1: submission order, kernel
// arguments, task-to-stream assignment, synchronisations) sits in device memory and
// persistent workgroups execute it themselves, so a dependent task starts as soon as a
// counter in memory says its producers are done, instead of after a round trip through
// the command processor. Streams keep the meaning they have in Section 2 ("GPU Streams"):
// each stream is served, in FIFO order, by its own gang of workgroups (picked on one XCD,
// so a stream's tensors stay in that XCD's L2); an event is a completion counter:
// recording = each workgroup of the producer adds 1 with release semantics after its
// tiles, waiting = polling until the counter reaches (workgroups of the producer) x
// (replay number), then dropping the compute unit's L1. A tensor that another XCD reads is
// stored and loaded with device-scope accesses, so no L2 is ever flushed or invalidated. Every wait is bounded: a workgroup that runs out of
// spins raises the error flag and every workgroup leaves.
// ------------------------------------------------------------------------------------
// One resident workgroup = kSubs sub-blocks of kBlock threads; the first `subs` of them take
// tile unit * subs + sub of every unit the workgroup owns (a task whose tiles keep the memory
// pipeline of a compute unit busy is better spread over more compute units: subs = 1). All
// sub-blocks walk the same number of units (tile functions may contain workgroup barriers):
// a sub-block without a tile calls the tile function with `live` false, which only takes
// part in the barriers.
// `words` points at the record's argument block in LDS; it is the same for every lane, so
// each word is moved into a scalar register.
template <int KID, class Wait>
__device__ __forceinline__ void run_tiles(const unsigned* words, int unit, int step, int ntiles, int subs, float* smem, int sub,
                                          int tid, bool fin, Wait& wait) {
    using A = typename KernelOf<KID>::Args;
    static_assert(sizeof(A) <= kArgWords * 4 && sizeof(A) % 4 == 0, "argument block does not fit the record");
    unsigned w[sizeof(A) / 4];
#pragma unroll
    for (size_t i = 0; i < sizeof(A) / 4; ++i) w[i] = __builtin_amdgcn_readfirstlane(words[i]);
    A a;
    __builtin_memcpy(&a, w, sizeof(A));
    const int nunits = (ntiles + subs - 1) / subs;
#define NG_LOOP(FI)                                                                  \
    for (; unit < nunits; unit += step) {                                            \
        const int tile = unit * subs + sub;                                          \
        const bool live = sub < subs && tile < ntiles;                               \
        KernelOf<KID>::template tile<FI>(a, live ? tile : 0, smem, tid, live, wait); \
    }
    if (!fin) { NG_LOOP(false) }
    else { NG_LOOP(true) }
#undef NG_LOOP
}

// The wait of one list entry for the completion counters of its parents; see NoWait for the
// contract. The first call does the work: lane j of the first wavefront polls parent j, then
// the compute unit's L1 is dropped and the workgroup meets at a barrier. Later calls (further
// tiles of the same entry) return at once.
// The polling loop of one lane.
// 0: the counter has reached the target; 1: it has not (`once`: after a single look, otherwise because
// another wait in the grid gave up); 2: ran out of spins.
__device__ __forceinline__ int spin_until(unsigned* counter, unsigned target, bool far, bool once, unsigned spin_limit,
                                                    int* error_dev, int poll_sleep) {
    unsigned spins = 0;
    for (;;) {
        unsigned seen;
        if (far) {
            seen = __hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            // read the counter where it lives, in this XCD's L2: a compare-and-swap that can
            // never match returns the current value (a plain load could be served by a stale
            // L1 line, and an atomic add of 0 is folded into such a load by the compiler)
            seen = 0xFFFFFFFFu;
            __hip_atomic_compare_exchange_strong(counter, &seen, 0xFFFFFFFFu, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        if ((int)(seen - target) >= 0) return 0;
        if (once) return 1;
        if (++spins > spin_limit) return 2;
        if ((spins & 63u) == 0 && __hip_atomic_load(error_dev, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return 1;
        if (poll_sleep == 0) __builtin_amdgcn_s_sleep(1);
        else if (poll_sleep == 1) __builtin_amdgcn_s_sleep(4);
        else __builtin_amdgcn_s_sleep(16);
    }
}

template <bool LATE>                 // LATE: the entry may have late parents (kernels with a fused add_n)
struct CounterWait {
    const DevPlan& plan;
    const unsigned* rec;             // the entry's record in LDS
    int* s_abort;
    int* s_late;                     // LDS flag: the late parents were already complete at the first wait
    unsigned epoch;
    int task, np, n_late, lane;      // np parents in all, the last n_late of them awaited by `late`
    unsigned long long* stamp;       // this entry's three clock readings when tracing, else nullptr (same for all lanes)
    bool pending, late_pending;
    bool far_out_;                   // the entry's results are stored with device-scope stores

    __device__ __forceinline__ bool far_out() const { return far_out_; }

    // Lane j of the first wavefront (first <= j < last) polls parent j until its counter has reached this
    // replay's target (`once`: looks a single time); true if it has. Other lanes return true.
    __device__ __forceinline__ bool poll(int first, int last, bool once) {
        bool ok = true;
        if (lane >= first && lane < last) {
            const unsigned target = rec[16 + lane] * epoch;
            const unsigned pw = rec[8 + lane];
            const bool far = (pw >> 31) != 0;
            unsigned* counter = (far ? plan.done : plan.done_near) + (size_t)(pw & 0x7fffffffu) * plan.done_stride;
            const int status = spin_until(counter, target, far, once, plan.spin_limit, plan.error_dev, plan.poll_sleep);
            ok = status == 0;
            if (status == 2) {
                atomicExch(plan.error_dev, task + 1);
                *plan.error_host = task + 1;
            }
        }
        return ok;
    }

    __device__ __forceinline__ void operator()() {
        if (!pending) return;
        pending = false;
        if (np > 0) {
            if (lane < 64) {                                    // first wavefront: lane j watches parent j
                const bool ok = poll(0, np - n_late, false);
                if (__any(!ok)) {
                    if (lane == 0) *s_abort = 1;
                }
                if (LATE && n_late > 0) {                       // usually the late parents are done as well by now
                    const bool there = poll(np - n_late, np, true);
                    const bool all_there = !__any(!there);
                    if (lane == 0) *s_late = all_there ? 1 : 0;
                }
                // Make the producers' stores visible to this compute unit. Producers on this
                // XCD have their results in the shared L2 already: dropping this CU's vector
                // L1 is enough (what a workgroup-scope acquire does when the waves of a
                // workgroup sit on different CUs). Tensors produced on another XCD are never
                // cached here at all: their loads are device-scope accesses (far_in).
                asm volatile("buffer_inv sc0" ::: "memory");
            }
            __syncthreads();                                    // also waits for the invalidate to finish
        }
        if (stamp != nullptr && lane == 0) stamp[1] = wall_clock64();
    }

    // Second wait of an entry whose tiles have a fused add_n: for the producers of the other operands.
    __device__ __forceinline__ void late() {
        if (!late_pending) return;
        late_pending = false;
        if (!LATE || n_late == 0 || *s_late != 0) return;       // same decision in every thread
        if (lane < 64) {
            const bool ok = poll(np - n_late, np, false);
            if (__any(!ok)) {
                if (lane == 0) *s_abort = 1;
            }
            asm volatile("buffer_inv sc0" ::: "memory");
        }
        __syncthreads();
    }
};

// BUILD selects which tile functions are compiled in (see in_build): the lean build leaves out the kernels
// that only large problems use - their register needs would otherwise shape the allocation of the whole
// replay kernel -, the train build has the lean kernels plus those of graphs that train.
template <int BUILD>
__global__ __launch_bounds__(kGroup) void resident_kernel(DevPlan plan, unsigned epoch) {
    constexpr int kSmemPerSub = BUILD == BUILD_FULL ? kSmemFloatsWide : kSmemFloats;
    __shared__ __align__(16) float smem_all[kSubs * kSmemPerSub];
    __shared__ uint4 recs[kRecordsInLds * (kRecordWords / 4)];
    __shared__ int s_abort, s_late;
    const int lane = threadIdx.x;
    const int sub = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kBlock), tid = (int)threadIdx.x % kBlock;
    float* smem = smem_all + sub * kSmemPerSub;
    if (lane == 0) s_abort = 0;
    const int e_begin = plan.wg_first[blockIdx.x], e_end = plan.wg_first[blockIdx.x + 1];
    // The plan keeps tensors in XCD-private L2s on the assumption that workgroups with equal index mod 8
    // share an XCD. Every launch checks it: each workgroup files its XCC id under its class together with
    // the replay number (a maximum, so whoever comes second in a class sees what the first one filed); the
    // answer is looked at when the workgroup is done, and a disagreement raises the error flag.
    unsigned long long xcc_prev = 0, xcc_mine = 0;
    if (plan.xcc_seen != nullptr && lane == 0) {
        xcc_mine = ((unsigned long long)epoch << 8) | (unsigned long long)(__builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)) & 15u);   // XCC_ID, bits 3:0
        xcc_prev = __hip_atomic_fetch_max(plan.xcc_seen + (blockIdx.x & 7), xcc_mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }

    for (int chunk = e_begin; chunk < e_end; chunk += kRecordsInLds) {
        // this workgroup's next records: global memory -> LDS, 16 bytes per lane and load
        const int count = min(kRecordsInLds, e_end - chunk);
        __syncthreads();                                        // the previous chunk is no longer read
        {
            const uint4* src = reinterpret_cast<const uint4*>(plan.records + chunk);
            for (int i = lane; i < count * (kRecordWords / 4); i += kGroup) recs[i] = src[i];
        }
        __syncthreads();
        for (int e = 0; e < count; ++e) {
            const unsigned* rec = reinterpret_cast<const unsigned*>(recs + e * (kRecordWords / 4));
            const int task = __builtin_amdgcn_readfirstlane(rec[0]), kid = __builtin_amdgcn_readfirstlane(rec[1]);
            const int ntiles = __builtin_amdgcn_readfirstlane(rec[2]), np = __builtin_amdgcn_readfirstlane(rec[3]);
            const int tile0 = __builtin_amdgcn_readfirstlane(rec[4]), step = __builtin_amdgcn_readfirstlane(rec[5]);
            const int flags = __builtin_amdgcn_readfirstlane(rec[6]), subs_word = __builtin_amdgcn_readfirstlane(rec[7]);
            const int subs = subs_word & 0xff, xcd_peers = subs_word >> 8;
            const bool far_in = (flags & 1) != 0, far_out = (flags & 2) != 0;
            const int n_late = (flags >> 8) & 0xff;
            // tracing: thread 0 stamps the clock into this entry's own slot (plain stores, nothing waits for them)
            unsigned long long* stamp = plan.trace != nullptr ? plan.trace + 3 * (size_t)(chunk + e) : nullptr;
            if (stamp != nullptr && lane == 0) stamp[0] = wall_clock64();
            // What the task can do without its inputs (addresses, weights) happens inside the tile
            // function before it calls `wait`; an entry that fails to wait in time still runs its
            // tiles (all accesses stay in bounds) and the workgroup leaves right after.
            // (every entry has at least one round of tiles, so the tile function always gets to call the wait)
            switch (kid) {
#define NG_CASE(KID)                                                                                                         \
    case KID:                                                                                                                \
        if constexpr (in_build(BUILD, KID)) {                                                                                \
            static_assert(smem_floats(KID) <= kSmemPerSub, "a sub-block has less LDS than the kernel takes");                \
            CounterWait<has_add_epilogue(KID)> wait{plan, rec, &s_abort, &s_late, epoch, task, np, n_late, lane, stamp, true, true, far_out}; \
            run_tiles<KID>(rec + 24, tile0, step, ntiles, subs, smem, sub, tid, far_in, wait);                               \
        }                                                                                                                    \
        break;
                NG_FOR_EACH_KID(NG_CASE)
#undef NG_CASE
                default: break;
            }
            // Publish protocol, step 1: every wave waits until all of its own vector memory operations have been
            // acknowledged (stores are counted by vmcnt on this target and a store is acknowledged by the level
            // its scope names: the XCD's L2 for a plain store through the write-through L1, the memory side for
            // an sc1 store). The barrier's own workgroup-scope fence does not include this wait. Step 2: the
            // barrier - every wave of the workgroup is past step 1. Step 3 (below): one lane bumps the counter,
            // an operation issued after the barrier and therefore after every acknowledgement.
            __builtin_amdgcn_s_waitcnt(0x0F70);                 // vmcnt(0), expcnt and lgkmcnt untouched
            __syncthreads();
            if (s_abort) return;
            if (stamp != nullptr && lane == 0) stamp[2] = wall_clock64();
            if (lane == 0) {
                // Publish completion. Readers on this XCD see the data in the shared L2 and are told through
                // a counter in that same L2 (an atomic without device scope is carried out there); if there
                // are readers elsewhere the tile functions have stored through to the memory side and the
                // device-scope counter is bumped as well.
                if (flags & 4)
                    __hip_atomic_fetch_add(plan.done_near + (size_t)task * plan.done_stride, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                bool tell_device = (flags & 8) != 0;
                if (flags & 16) {
                    // two levels: count the workgroups of this XCD in its L2; only the last one goes on
                    const unsigned before = __hip_atomic_fetch_add(plan.done_xcd + ((size_t)task * 8 + (blockIdx.x & 7)) * plan.done_stride, 1u,
                                                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    tell_device = before + 1u == epoch * (unsigned)xcd_peers;
                }
                if (tell_device)
                    __hip_atomic_fetch_add(plan.done + (size_t)task * plan.done_stride, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    if (plan.xcc_seen != nullptr && lane == 0 && (xcc_prev >> 8) == (xcc_mine >> 8) && (xcc_prev & 255u) != (xcc_mine & 255u)) {
        atomicExch(plan.error_dev, kErrorXcdMapping);
        *plan.error_host = kErrorXcdMapping;
    }
}

}  // namespace

template <> const void* resident_build_handle<NG_RESIDENT_BUILD>() { return reinterpret_cast<const void*>(&resident_kernel<NG_RESIDENT_BUILD>); }

}  // namespace ng
