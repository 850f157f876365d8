// Several independent tasks of one kernel in one launch (single-stream replay modes).
//
// Nimble (arXiv 2012.02732), Section 4.2, runs independent tasks of a network side by side on several streams. On this GPU a
// second stream costs a hand-over through the command processor per crossing, more than most of these tasks take; tasks of the
// same kernel need no second stream: their workgroups go out in one launch, which costs one launch gap and one tail instead
// of one of each per task. The kernels are those of the tasks themselves (one instantiation per kernel id, so nothing is shared
// with other kernels' registers); a workgroup finds its task by its index and takes that task's argument block from the kernel
// arguments with uniform loads. Launches and time of a replay, one task at a time -> gathered: training step of a NAS cell, batch 32
// 132 -> 62, 1049 -> 817 us, batch 96 2107 -> 1812 us, ten images of 27 x 27 635 -> 400 us; Inception-style network at batch 1
// 92 -> 56, 719 -> 585 us, six images 103 -> 65, 1148 -> 1039 us. The order this takes is that of plan_single_launches.
#include "ng_kernels.hip"

namespace ng {
namespace {

template <int KID>
__device__ __forceinline__ void gathered_tile(const GatherArgs<typename KernelOf<KID>::Args>& p, float* smem) {
    int place = (int)blockIdx.x, column = -1;
    if constexpr (is_pw_columns(KID)) {
        if (p.eights > 0) {
            const XcdShare s = xcd_share(place, p.end[kGatherMax - 1]);
            place = s.row, column = s.column;
        }
    }
    int which = 0, first = 0;
#pragma unroll
    for (int i = 0; i + 1 < kGatherMax; ++i)
        if (place >= p.end[i]) which = i + 1, first = p.end[i];
    const typename KernelOf<KID>::Args a = p.task[which];
    int tile = place - first;
    if constexpr (is_pw_columns(KID)) {
        if (column >= a.tiles_n) return;                        // the whole workgroup
        if (column >= 0) tile = is_pw_patch(KID) ? column * a.mtiles + tile : tile * a.tiles_n + column;
    }
    NoWait wait;
    KernelOf<KID>::template tile<false>(a, tile, smem, threadIdx.x, true, wait);
}
template <int KID>
__global__ __launch_bounds__(kBlock, min_waves(KID)) void gathered_kernel(GatherArgs<typename KernelOf<KID>::Args> p) {
    __shared__ __align__(16) float smem[smem_floats(KID)];
    gathered_tile<KID>(p, smem);
}
// With the device's clock read around it, as timed_kernel does.
template <int KID>
__global__ __launch_bounds__(kBlock, min_waves(KID)) void timed_gathered_kernel(GatherArgs<typename KernelOf<KID>::Args> p, unsigned long long* stamps) {
    __shared__ __align__(16) float smem[smem_floats(KID)];
    unsigned long long t0 = 0;
    if (threadIdx.x == 0) t0 = wall_clock64();
    gathered_tile<KID>(p, smem);
    __builtin_amdgcn_s_waitcnt(0x0F70);                          // vmcnt(0): this wave's stores are acknowledged
    __syncthreads();
    if (threadIdx.x == 0) {
        stamps[2 * (size_t)blockIdx.x] = t0;
        stamps[2 * (size_t)blockIdx.x + 1] = wall_clock64();
    }
}

// the kernels that a network runs several of side by side
#define NG_FOR_EACH_GATHERED(X)                                                                                         \
    X(KID_BN) X(KID_BN_V4) X(KID_ADD) X(KID_ADD_V4) X(KID_CONCAT) X(KID_CONCAT_V4) X(KID_POOL) X(KID_POOL_ROW_S1)       \
    X(KID_POOL_ROW_S2) X(KID_DW_K3S1) X(KID_DW_K3S2) X(KID_DW_K5S1) X(KID_DW_K5S2) X(KID_DW_LDS)                        \
    X(KID_PW_D4) X(KID_PW_D8) X(KID_PW_D16) X(KID_PW_64) X(KID_PW_V1) X(KID_PW_V2) X(KID_PW_V3) X(KID_PW_V4)            \
    X(KID_PW_S1) X(KID_PW_S2) X(KID_PW_S3) X(KID_PW_S4) X(KID_PW_P32) X(KID_PW_P64)                                     \
    X(KID_C3_M1) X(KID_C3_M2) X(KID_C3_M3) X(KID_C3_M4) X(KID_C3_L32) X(KID_C3_L64)                                     \
    X(KID_C3_P64) X(KID_C3_P96) X(KID_C3_Q32) X(KID_C3_Q64) X(KID_C3_Q128) X(KID_C3_R32) X(KID_C3_R128) X(KID_C3_SK)     \
    X(KID_PW_PX_FWD) X(KID_BN_RAW) X(KID_BN_BACKWARD) X(KID_PAIR_DW) X(KID_PAIR_DW_LDS) X(KID_PAIR_PW16)                \
    X(KID_PAIR_PW32) X(KID_POOL_DGRAD) X(KID_POOL_DGRAD_LDS) X(KID_SLICE_PAD) X(KID_SMALL_GEMM)

// conv1x1 from this many column blocks on: they are dealt out to the XCDs (xcd_share). In the tiles' own order the row tiles of a
// column block run on up to 8 XCDs and each of those reads the block into its own L2. Dealt out, the launches of 64 x 64 tiles of the
// Inception-style network at batch 32 read 1.58 GB from memory (12 launches; 1.88 in 34 of one task each in their own order). Four layers from 768 channels of
// 17 x 17 in one launch 94 -> 85 us, three of 288 channels and 35 x 35 60 -> 55; the whole network 3585 -> 3545 us. With fewer
// column blocks eight of them are too coarse a unit: 19 blocks are three for some XCDs and two for others.
constexpr int kXcdColumns = 32;
constexpr long kMaxWorkgroups = (1L << 32) / kBlock;            // a launch has fewer than 2^32 work items

template <int KID>
void fill(const std::vector<const Task*>& tasks, SingleLaunch& out) {
    GatherArgs<typename KernelOf<KID>::Args> p{};
    const int n = (int)tasks.size();
    for (int i = 0; i < n; ++i) std::memcpy(&p.task[i], tasks[i]->args, sizeof p.task[i]);
    if constexpr (is_pw_columns(KID)) {
        bool same = true;
        for (int i = 1; i < n; ++i) same = same && p.task[i].tiles_n == p.task[0].tiles_n;
        long rows = 0;
        for (int i = 0; i < n; ++i) rows += p.task[i].mtiles;
        if (same && p.task[0].tiles_n >= kXcdColumns && (p.task[0].tiles_n + 7L) / 8 * 8 * rows < kMaxWorkgroups) p.eights = (p.task[0].tiles_n + 7) / 8;
    }
    long total = 0;
    for (int i = 0; i < kGatherMax; ++i) {
        if constexpr (is_pw_columns(KID)) {
            if (i < n && p.eights > 0) { p.end[i] = (int)(total += p.task[i].mtiles); continue; }
        }
        if (i < n) total += tasks[i]->ntiles;
        p.end[i] = (int)total;
    }
    if (p.eights > 0) total *= 8L * p.eights;
    else if (n == 1) return;                                    // launched as it is
    if (total <= 0 || total >= kMaxWorkgroups) return;
    out.fn = reinterpret_cast<const void*>(&gathered_kernel<KID>);
    out.timed_fn = reinterpret_cast<const void*>(&timed_gathered_kernel<KID>);
    out.grid = (unsigned)total;
    out.args.resize(sizeof p);
    std::memcpy(out.args.data(), &p, sizeof p);
}

}  // namespace

bool can_gather(int kid) {
    switch (kid) {
#define NG_CASE(KID) case KID:
        NG_FOR_EACH_GATHERED(NG_CASE)
#undef NG_CASE
            return true;
        default: return false;
    }
}

// The launch that carries out `tasks`: one task as it is (unless its column blocks are dealt out to the XCDs), several of one kernel
// by that kernel's gathered form.
void make_gathered_launch(const std::vector<const Task*>& tasks, SingleLaunch& out) {
    out = SingleLaunch();
    for (const Task* t : tasks)
        if (t->kid != tasks[0]->kid || !t->fn) return;
    if (tasks.size() == 1) {
        const Task& t = *tasks[0];
        out.fn = t.fn, out.timed_fn = timed_kernel_handle(t.kid), out.grid = t.grid[0], out.lds_bytes = t.lds_bytes;
        out.args.assign(t.args, t.args + sizeof t.args);
        if (!is_pw_columns(t.kid)) return;
    }
    switch (tasks[0]->kid) {
#define NG_CASE(KID) case KID: fill<KID>(tasks, out); break;
        NG_FOR_EACH_GATHERED(NG_CASE)
#undef NG_CASE
        default: break;
    }
}

}  // namespace ng
