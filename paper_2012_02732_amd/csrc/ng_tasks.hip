// Stand-alone kernels (one per tile function), the kernels that repack weights at bind time, and the task table: which kernel
// a node gets, decided from its shapes.
#include "ng_kernels.hip"

namespace ng {
namespace {

// Batch-norm parameters -> one multiplier and one offset per channel, once, at bind time.
__global__ __launch_bounds__(kBlock) void fold_bn_kernel(const float* gamma, const float* beta, const float* mean,
                                                         const float* var, float eps, float* scale, float* shift, int C) {
    const int c = blockIdx.x * kBlock + threadIdx.x;
    if (c >= C) return;
    const float s = gamma[c] / sqrtf(var[c] + eps);
    scale[c] = s;
    shift[c] = beta[c] - mean[c] * s;
}

// The weights of both patch-stationary kernels, W[Cout][Cin][TAPS]: -> [block * TAPS + tap][Mf][part][lane][8 bf16], block = 16
// input channels, Mf = fragments of 32 rows; lane (r, g) holds row r, channels 8 g .. 8 g + 7; zero where m >= Cout.
// One thread per (slice, fragment, lane).
__global__ __launch_bounds__(kBlock) void pack_split_weights_kernel(const float* w, float* wq, int Cout, int Cin, int taps, int Mf, long total) {
    const long idx = (long)blockIdx.x * kBlock + threadIdx.x;
    if (idx >= total) return;
    const int lane = (int)(idx & 63);
    const long f = idx >> 6;
    const int mf = (int)(f % Mf), slice = (int)(f / Mf), block = slice / taps, tap = slice - block * taps;
    const int m = mf * 32 + (lane & 31), c = block * 16 + 8 * (lane >> 5);
    float v[8];
    for (int q = 0; q < 8; ++q) v[q] = m < Cout && c + q < Cin ? w[((size_t)m * Cin + c + q) * taps + tap] : 0.f;
    u32x4 part[3];
    split8(v, part);
    for (int p = 0; p < 3; ++p) reinterpret_cast<u32x4*>(wq)[(f * 3 + p) * 64 + lane] = part[p];
}

// W[Cout][Cin] -> W^T[CinP][CoutP], zero where k >= Cin or m >= Cout
__global__ __launch_bounds__(kBlock) void pack_pw_lds_weights_kernel(const float* w, float* wp, int Cout, int Cin, int CoutP, long total) {
    const long idx = (long)blockIdx.x * kBlock + threadIdx.x;
    if (idx >= total) return;
    const int m = (int)(idx % CoutP), k = (int)(idx / CoutP);
    wp[idx] = (m < Cout && k < Cin) ? w[(size_t)m * Cin + k] : 0.f;
}

// W[Cout][Cin][3][3] -> W'^T[tap * CinP + ci][CoutP], zero where ci >= Cin or m >= Cout
__global__ __launch_bounds__(kBlock) void pack_c3_lds_weights_kernel(const float* w, float* wp, int Cout, int Cin, int CinP, int CoutP, long total) {
    const long idx = (long)blockIdx.x * kBlock + threadIdx.x;
    if (idx >= total) return;
    const int m = (int)(idx % CoutP);
    const int k = (int)(idx / CoutP);
    const int tap = k / CinP, ci = k - tap * CinP;
    wp[idx] = (m < Cout && ci < Cin) ? w[((size_t)m * Cin + ci) * 9 + tap] : 0.f;
}

__global__ __launch_bounds__(kBlock) void pack_pw_weights_kernel(const float* w, float* wp, int Cout, int Cin,
                                                                  int ksteps, int total) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= total) return;
    const int l = i & 63, blk = i >> 6;
    const int ks = blk % ksteps, rt = blk / ksteps;
    const int m = rt * 16 + (l & 15), k = ks * 4 + (l >> 4);
    wp[i] = (m < Cout && k < Cin) ? w[(size_t)m * Cin + k] : 0.f;
}

__global__ __launch_bounds__(kBlock) void pack_pw_weights_k4_kernel(const float* w, float* wp, int Cout, int Cin,
                                                                     int groups, int total) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= total) return;
    const int q = i & 3, l = (i >> 2) & 63, blk = i >> 8;
    const int gi = blk % groups, rt = blk / groups;
    const int m = rt * 16 + (l & 15), k = 16 * gi + 4 * q + (l >> 4);
    wp[i] = (m < Cout && k < Cin) ? w[(size_t)m * Cin + k] : 0.f;
}
// Stand-alone kernel of one tile function: one workgroup per tile.
template <int KID>
__global__ __launch_bounds__(kBlock, min_waves(KID)) void standalone_kernel(typename KernelOf<KID>::Args a) {
    __shared__ __align__(16) float smem[smem_floats(KID)];
    NoWait wait;
    KernelOf<KID>::template tile<false>(a, blockIdx.x, smem, threadIdx.x, true, wait);
}

// The same, with the device's clock read around it: workgroup b leaves in stamps[2 b] the time of its
// first instruction and in stamps[2 b + 1] the time at which all its stores were acknowledged (100 MHz
// constant clock; plain stores, one pair per workgroup, so the readings do not disturb each other). The
// latest end minus the earliest start is the time the GPU is busy with the task when it runs alone,
// without what the command processor spends around a dispatch.
template <int KID>
__global__ __launch_bounds__(kBlock, min_waves(KID)) void timed_kernel(typename KernelOf<KID>::Args a, unsigned long long* stamps) {
    __shared__ __align__(16) float smem[smem_floats(KID)];
    unsigned long long t0 = 0;
    if (threadIdx.x == 0) t0 = wall_clock64();
    NoWait wait;
    KernelOf<KID>::template tile<false>(a, blockIdx.x, smem, threadIdx.x, true, wait);
    __builtin_amdgcn_s_waitcnt(0x0F70);                          // vmcnt(0): this wave's stores are acknowledged
    __syncthreads();
    if (threadIdx.x == 0) {
        stamps[2 * (size_t)blockIdx.x] = t0;
        stamps[2 * (size_t)blockIdx.x + 1] = wall_clock64();
    }
}

// ------------------------------------------------------------------------------------
// task construction
// ------------------------------------------------------------------------------------
template <int KID>
void set_kernel(Task& t, const typename KernelOf<KID>::Args& a, long ntiles) {
    using A = typename KernelOf<KID>::Args;
    static_assert(sizeof(A) <= kLaunchArgBytes, "argument block too large");
    static_assert(std::is_trivially_copyable<A>::value, "argument block must be plain data");
    t.kid = KID;
    t.fn = reinterpret_cast<const void*>(&standalone_kernel<KID>);
    t.name = KernelOf<KID>::name;
    std::memcpy(t.args, &a, sizeof(A));
    t.args_bytes = sizeof(A);
    t.ntiles = ntiles;
    t.grid[0] = (unsigned)ntiles;
}

long ceil_div(long a, long b) { return (a + b - 1) / b; }

// conv1x1 forward / input gradient of a graph that trains: the kernel that reads pixels 128 bits at a time re-reads the
// activations once per 16 rows, which pays while the rows are few (the 64 x 64 LDS-staged GEMM tile otherwise).
bool pw_px_applies(const GemmArgs& a) {
    const long hw = (long)a.Ho * a.Wo;
    return hw >= 4 && a.K % 4 == 0 && a.M <= 256 && a.bias == nullptr && (long)a.K * a.N * 4 < (1L << 31) &&
           (long)a.M * a.N * 4 < (1L << 31);
}
// The classifier's GEMMs (1 x 1 maps, a few thousand outputs, K up to a few hundred): no tiles. K over the lanes of a
// wavefront where both operands run along k and K is long, else a thread per output.
constexpr long kSmallGemmOutputs = 1 << 16, kSmallGemmK = 1024;
void set_small_gemm(Task& t, SmallGemmArgs a, void (*set)(Task&, const SmallGemmArgs&, long)) {
    a.by_wave = a.sak == 1 && a.sbk == 1 && a.K >= 64;
    set(t, a, a.by_wave ? ceil_div((long)a.M * a.N, kBlock / 64) : ceil_div((long)a.M * a.N, kBlock));
}
long pw_px_tiles(const GemmArgs& a) {
    const long hw = (long)a.Ho * a.Wo;
    return ceil_div(ceil_div(a.N / hw * ceil_div(hw, 4), 16) * ceil_div(a.M, 16), 4);
}
// Backward kernels whose ragged edges (planes or rows that are no multiple of 16 or 4 pixels) cost extra work per edge: below
// this many pixels (weight gradients) or elements (depthwise input gradient) a task is a few workgroups that wait for
// memory once either way, and the general kernels stay. Above it, a training step of a NAS cell: 36 channels, 10 images of
// 27 x 27 pixels 1090 -> 750 us; 24 channels, 60 images of 30 x 30 pixels 2945 -> 1225 us.
constexpr long kRaggedMinPixels = 1024, kRaggedMinElements = 1 << 16;

// Direct conv1x1: k steps per chunk by problem depth, and the padded step count of the packed copy.
int pw_chunk(long cin) { return cin <= 64 ? 4 : (cin <= 128 ? 8 : 16); }
int pw_padded_steps(long cin) {
    const long unit = 4L * pw_chunk(cin);
    return (int)(ceil_div(ceil_div(cin, 4), unit) * unit);
}

}  // namespace

// Which XCD runs workgroup i? The planner relies on workgroups with equal i mod 8 sharing one
// (a 1-D grid is dealt out round-robin on this GPU); the runtime checks it with this probe
// before it trusts XCD-local L2s.
namespace {
__global__ __launch_bounds__(kGroup) void xcd_probe_kernel(int* xcd_of_workgroup) {
    if (threadIdx.x == 0) xcd_of_workgroup[blockIdx.x] = (int)__builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11));   // XCC_ID, bits 3:0
}
}  // namespace
const void* xcd_probe_kernel_handle() { return reinterpret_cast<const void*>(&xcd_probe_kernel); }

// Where the partial results of a weight-gradient task are (kind PARTS_NONE: it has none, it writes the gradient itself), and
// the same task with its sum left to a later launch.
SgdTile gradient_parts(const Task& t) {
    SgdTile p{};
    switch (t.kid) {
        case KID_GEMM_PW_WGRAD: case KID_GEMM_C3_WGRAD: case KID_PW_WGRAD_PX: case KID_PW_WGRAD_PX2: case KID_C3_WGRAD_PX: case KID_C3_WGRAD_PX2: {
            GemmArgs a;
            std::memcpy(&a, t.args, sizeof a);
            if (a.splits <= 1) break;
            p.kind = PARTS_BLOCKS, p.parts = a.ws, p.splits = a.splits, p.width = a.N, p.blocks = a.tiles_n;
            p.edge = (t.kid == KID_GEMM_PW_WGRAD || t.kid == KID_GEMM_C3_WGRAD) ? kGemmTile : (t.kid == KID_PW_WGRAD_PX || t.kid == KID_C3_WGRAD_PX) ? 16 : 32;
            break;
        }
        case KID_DW_WGRAD: {
            DwGradArgs a;
            std::memcpy(&a, t.args, sizeof a);
            if (a.chunks > 1) p.kind = PARTS_PLANES, p.parts = a.ws, p.splits = a.chunks, p.width = a.K * a.K;
            break;
        }
        case KID_BN_WGRAD: {
            BnRawArgs a;
            std::memcpy(&a, t.args, sizeof a);
            if (a.chunks > 1) p.kind = PARTS_PAIRS, p.parts = a.ws, p.splits = a.chunks, p.width = a.C;
            break;
        }
        default: break;
    }
    return p;
}
void leave_sum_to_later_launch(Task& t) {
    if (t.kid == KID_DW_WGRAD) reinterpret_cast<DwGradArgs*>(t.args)->cnt = nullptr;
    else if (t.kid == KID_BN_WGRAD) reinterpret_cast<BnRawArgs*>(t.args)->cnt = nullptr;
    else reinterpret_cast<GemmArgs*>(t.args)->cnt = nullptr;
}

// The launch that carries out the update nodes `members` (their stand-alone tasks in `tasks`) at once; in_parts[v] != 0:
// gradient node v is left in parts. The shares of the members are appended to `table`, the host copy of the device
// table that will sit at `table_dev`: the task's argument points at its first share there.
void make_sgd_batch_task(const ng_graph* g, const std::vector<Task>& tasks, const std::vector<int>& members, const std::vector<char>& in_parts,
                         std::vector<SgdTile>& table, const SgdTile* table_dev, Task& t) {
    const size_t first = table.size();
    for (int v : members) {
        SgdArgs a;
        std::memcpy(&a, tasks[v].args, sizeof a);
        const int gradient = g->nodes[v].preds[0];
        const bool parts = in_parts[gradient] != 0;
        const int per = parts ? kSgdSumElems : kSgdTileElems;
        for (int at = 0; at < a.total || at == 0; at += per) {
            SgdTile s = parts ? gradient_parts(tasks[gradient]) : SgdTile{};
            s.w = a.w + at, s.g = const_cast<float*>(a.g) + a.offset + at, s.flag = at == 0 ? a.flag : nullptr, s.lr = a.lr;
            s.count = std::min(a.total - at, per), s.first = a.offset + at;
            table.push_back(s);
        }
    }
    t = Task();
    t.block[0] = kBlock;
    set_kernel<KID_SGD_BATCH>(t, SgdBatchArgs{table_dev + first}, (long)(table.size() - first));
}

// Which two stand-alone kernels have a launch of their own together (pair_tile): input gradient first, weight gradient second.
static int pair_kid(const Task& first, const Task& second) {
    const int kid_first = first.kid, kid_second = second.kid;
    if (kid_first == KID_DW_DGRAD && kid_second == KID_DW_WGRAD) return KID_PAIR_DW;
    if (kid_first == KID_DW_DGRAD_LDS && kid_second == KID_DW_WGRAD)
        return dw_wgrad_by_quads(*reinterpret_cast<const DwGradArgs*>(second.args)) ? KID_PAIR_DW_LDS : KID_NONE;
    if (kid_first == KID_PW_PX_DGRAD && kid_second == KID_PW_WGRAD_PX) return KID_PAIR_PW16;
    if (kid_first == KID_PW_PX_DGRAD && kid_second == KID_PW_WGRAD_PX2) return KID_PAIR_PW32;
    return KID_NONE;
}
bool can_pair(const Task& first, const Task& second) { return pair_kid(first, second) != KID_NONE; }
// The kernel of the launch of task v with everything that rides on it (`fused_into` as decided).
int launch_kid(const std::vector<Task>& tasks, const std::vector<int>& fused_into, int v) {
    for (size_t w = 0; w < tasks.size(); ++w) {
        if (fused_into[w] != v || (int)w == v) continue;
        const int a = tasks[v].kid, b = tasks[w].kid;
        if (b == KID_SGD) return KID_SGD_BATCH;
        if ((a == KID_BN_DGRAD && b == KID_BN_WGRAD) || (a == KID_BN_WGRAD && b == KID_BN_DGRAD)) return KID_BN_BACKWARD;
        if (can_pair(tasks[v], tasks[w])) return pair_kid(tasks[v], tasks[w]);
        if (can_pair(tasks[w], tasks[v])) return pair_kid(tasks[w], tasks[v]);
    }
    return tasks[v].kid;
}
template <int KID>
static void set_pair(const Task& first, const Task& second, Task& t) {
    typename KernelOf<KID>::Args p{};
    std::memcpy(&p.a, first.args, sizeof p.a);
    std::memcpy(&p.b, second.args, sizeof p.b);
    p.na = (int)first.ntiles, p.nb = (int)second.ntiles;
    t = Task();
    t.block[0] = kBlock;
    set_kernel<KID>(t, p, first.ntiles + second.ntiles);
}
template <int KID>
static void set_pw_backward(const Task& dgrad, const Task& wgrad, Task& t) {
    PairPwArgs p{};
    std::memcpy(&p.a, dgrad.args, sizeof p.a);
    std::memcpy(&p.b, wgrad.args, sizeof p.b);
    const long hw = (long)p.a.Ho * p.a.Wo, groups = ceil_div(p.a.N / hw * ceil_div(hw, 4), 16);
    p.na = (int)ceil_div((p.b.splits >= kXcdSplits ? ceil_div(groups, p.b.splits) : groups) * ceil_div(p.a.M, 16), 4);
    p.nb = (int)(wgrad.ntiles / p.b.splits);
    t = Task();
    t.block[0] = kBlock;
    set_kernel<KID>(t, p, pw_backward_tiles(p.na, p.nb, p.b.splits));
}
void make_pair_task(const Task& first, const Task& second, Task& t) {
    switch (pair_kid(first, second)) {
        case KID_PAIR_DW: set_pair<KID_PAIR_DW>(first, second, t); break;
        case KID_PAIR_DW_LDS: set_pair<KID_PAIR_DW_LDS>(first, second, t); break;
        case KID_PAIR_PW16: set_pw_backward<KID_PAIR_PW16>(first, second, t); break;
        case KID_PAIR_PW32: set_pw_backward<KID_PAIR_PW32>(first, second, t); break;
        default: t = first; break;
    }
}

// The launch that computes a batch-norm's parameter gradients (task `wgrad`) and its input gradient (task `dgrad`, same
// dy, x and parameters) in one walk over dy and x.
void make_bn_backward_task(const Task& dgrad, const Task& wgrad, Task& t) {
    BnRawArgs a, d;
    std::memcpy(&a, wgrad.args, sizeof a);
    std::memcpy(&d, dgrad.args, sizeof d);
    a.dx = d.y;
    t = Task();
    t.block[0] = kBlock;
    set_kernel<KID_BN_BACKWARD>(t, a, wgrad.ntiles);
}

template <> const void* resident_build_handle<BUILD_LEAN>();
template <> const void* resident_build_handle<BUILD_FULL>();
template <> const void* resident_build_handle<BUILD_TRAIN>();
const void* resident_kernel_handle(int build) {
    return build == BUILD_TRAIN ? resident_build_handle<BUILD_TRAIN>() : build == BUILD_FULL ? resident_build_handle<BUILD_FULL>() : resident_build_handle<BUILD_LEAN>();
}

namespace {
__global__ void empty_kernel() {}
}  // namespace
const void* empty_kernel_handle() { return reinterpret_cast<const void*>(&empty_kernel); }

// The stand-alone kernel of a kernel id (nullptr if the id has none) and its name: lets the runtime
// launch a task in the variant a replay mode really executes (e.g. a convolution with its fused
// batch-norm and add_n), by itself, for timing.
const void* standalone_kernel_handle(int kid, const char** name) {
    switch (kid) {
#define NG_HANDLE(KID) \
    case KID:          \
        if (name) *name = KernelOf<KID>::name; \
        return reinterpret_cast<const void*>(&standalone_kernel<KID>);
        NG_FOR_EACH_KID(NG_HANDLE)
#undef NG_HANDLE
        default: return nullptr;
    }
}
const void* timed_kernel_handle(int kid) {
    switch (kid) {
#define NG_HANDLE(KID) \
    case KID: return reinterpret_cast<const void*>(&timed_kernel<KID>);
        NG_FOR_EACH_KID(NG_HANDLE)
#undef NG_HANDLE
        default: return nullptr;
    }
}

namespace {
// Which conv1x1 kernel a node gets. Decided from shapes alone, so that the size of the
// repacked weights is known before any memory is bound.
struct PwChoice {
    enum Kind { NONE, GEMV, LDS64, DIRECT32, K4_VEC, K4_WORD, C3_LDS, C3_PATCH, PW_PATCH } kind = NONE;
    int kid = KID_NONE;       // C3_PATCH, PW_PATCH: which of the kernels
    int in_flight = 0;        // K4: groups of 4 k-steps in flight (1..4); DIRECT32: k-steps per chunk
    int groups = 0;           // K4: groups in the packed copy (a multiple of 4 * in_flight); DIRECT32: padded k-steps
    size_t packed = 0;        // floats of repacked weights
};
// K split of the 16-row kernels: groups of 4 k-steps, padded so that every wavefront gets
// the same whole number of chunks of `in_flight` groups.
void k4_split(long k_total, long cout, PwChoice& c) {
    const long groups = ceil_div(ceil_div(k_total, 4), 4);
    long gw = ceil_div(groups, 4);                           // groups per wavefront
    if (gw <= 4) {
        c.in_flight = (int)gw;
    } else {
        const long pad3 = ceil_div(gw, 3) * 3, pad4 = ceil_div(gw, 4) * 4;
        c.in_flight = pad3 < pad4 ? 3 : 4;
        gw = std::min(pad3, pad4);
    }
    c.groups = (int)(4 * gw);
    c.packed = (size_t)((cout + 15) / 16) * c.groups * 256;
}
constexpr long kPwPatchMinCols = 2048;
constexpr long kPoolRowMinOutputs = 1 << 20;   // pool3x3: from here on the kernel with four outputs of a column per thread
constexpr long kDwLdsMinOutputs = 1 << 18;     // dwconv: from here on whole planes through LDS (dwconv_lds), where the planes allow
PwChoice choose_pw(const ng_graph* g, int v) {
    PwChoice c;
    const Node& nd = g->nodes[v];
    if (nd.op != NG_OP_CONV1X1 && nd.op != NG_OP_FC) return c;
    const Shape& o = nd.out;
    const long cin = g->nodes[nd.preds[0]].out.c;
    const long hw = o.h * o.w, cols = o.n * hw;
    if (nd.op == NG_OP_FC && o.n <= 8) { c.kind = PwChoice::GEMV; return c; }
    // many output pixels, whole blocks of 16 input channels: activations pixel-major in LDS, weights straight from memory;
    // 64-row tiles unless that leaves most compute units without one
    const long tiles64 = ((o.c + 63) / 64) * ((cols + 63) / 64);
    if (cols >= kPwPatchMinCols && cin % 16 == 0 && cin >= 64 && tiles64 >= 64 && cols * cin * 4 < (1L << 31) && cin * (o.c + 63) * 6 < (1L << 31) && !knob("NG_NO_PATCH_KERNELS")) {
        c.kind = PwChoice::PW_PATCH;
        c.kid = tiles64 < 200 ? KID_PW_P32 : KID_PW_P64;
        const long tm = c.kid == KID_PW_P32 ? 32 : 64;
        c.groups = (int)cin;
        c.packed = (size_t)cin * (size_t)((o.c + tm - 1) / tm * tm) * 3 / 2;   // [Cin / 16][CoutP / 32][3 parts][64 lanes][8 bf16]
        return c;
    }
    // large problems (many 64 x 64 tiles) keep the LDS-tiled throughput kernel
    if (((o.c + 63) / 64) * ((cols + 63) / 64) >= 256) {
        c.kind = PwChoice::LDS64;
        c.groups = (int)((cin + 15) / 16 * 16);                              // CinP: whole K slices of 16
        c.packed = (size_t)c.groups * (size_t)((o.c + 63) / 64 * 64);       // W^T[CinP][CoutP]
        return c;
    }
    const bool vec = hw % 4 == 0;
    const long tiles16 = ((o.c + 15) / 16) * ((cols + 15) / 16);
    // Maps without 128-bit loads: the 16 x 16 tiles with K split over the wavefronts up to 512 of them (two workgroups per
    // compute unit), 32 x 32 tiles, which read less, beyond. The 32 x 32 kernels hold registers that only the full build of
    // the resident kernel has room for: a NAS cell on 25 x 25 maps (240 tiles) replays in 356 us with 16 x 16 tiles (lean
    // build) and in 474 us with two of its tasks on 32 x 32 tiles, which take 4.2 us there against 2.9 us; an
    // Inception-style network at batch 1 (31 layers of 17 x 17 and 35 x 35 maps, 228 - 385 tiles) 765 against 810 us.
    // Graphs in the full build and launched ones gain as well: of chains of twelve layers between 44 - 2048 channels, 7 x 7 to 45 x 45
    // (121 - 512 tiles), 17 of 17 are faster as a single-stream graph and 15 in the resident kernel (two 2 % slower): 17 x 17 768 <-> 192 86 / 175 -> 63 / 123 us, 35 x 35
    // 64 <-> 64 46 / 80 -> 42 / 46, 7 x 7 2048 <-> 1000 162 / 350 -> 103 / 115, 35 x 35 1024 <-> 64 120 / 197 -> 113 / 183.
    if (!vec && tiles16 > 512) {
        c.kind = PwChoice::DIRECT32;
        c.in_flight = pw_chunk(cin);
        c.groups = pw_padded_steps(cin);
        c.packed = (size_t)((o.c + 15) / 16) * 64 * c.groups;
        return c;
    }
    c.kind = vec ? PwChoice::K4_VEC : PwChoice::K4_WORD;
    k4_split(cin, o.c, c);
    return c;
}
// conv3x3 with at least 8 input channels runs as an implicit GEMM with K = 9 Cin
constexpr long kC3LdsMinCols = 2048;      // measured: below this the 16 x 16 tiles (more workgroups, shorter K loops each) win
// The patch-stationary kernels: rows and pixels of a tile; a tile's time while the chip is full of them (64: one of 64 x 64), from 430
// layers of 9 x 9 to 130 x 130, 16 - 384 output channels, strides of 1 and 2: choose_patch_kernel takes the fastest of the kernels, or one
// within 5 % of it.
struct PatchKernel { int kid, tm, tn; double cost; };
constexpr PatchKernel kPatchKernels[] = {{KID_C3_P64, 64, 64, 64}, {KID_C3_P96, 96, 64, 94}, {KID_C3_Q32, 32, 128, 68},
                                         {KID_C3_Q64, 64, 64, 73}, {KID_C3_Q128, 64, 128, 117}, {KID_C3_R32, 32, 128, 74},
                                         {KID_C3_R128, 64, 128, 140}, {KID_C3_SK, 32, 32, 0}};
// Largest patch a run of tn consecutive output pixels can need: the rows it touches (a run can start at the end of a
// row), stride apart, plus two, each W + 2 pad wide.
long patch_pixels(long tn, long W, long Ho, long Wo, long stride, long pad) {
    const long rows = std::min(Ho, (tn - 2) / Wo + 2);
    return ((rows - 1) * stride + 3) * (W + 2 * pad);
}
// The strips that an image is cut into, so that the patch of every run of tn pixels of a strip fits into the kernel's LDS: the width
// of all but the last (0: none fits) and the runs of an image. As few strips as possible, unless more of them save more than one run in 33.
struct Strips { long width, runs; };
long largest_patch(long tn, long width, long Ho, long stride) {              // as the kernel counts it, over the runs of one strip
    long most = 0;
    const long row = (width - 1) * stride + 3, pixels = width * Ho;
    auto run = [&](long p) {
        const long last = std::min(p + tn, pixels) - 1;
        most = std::max(most, ((last / width - p / width) * stride + 2) * row + last % width * stride + 3 - p % width * stride);
    };
    // a whole run's patch depends on the column it starts in, and those repeat after at most `width` runs; the last run may be short
    for (long i = 0, start = 0; i < width && start < pixels; ++i, start += tn) run(start);
    run((pixels - 1) / tn * tn);
    return most;
}
Strips choose_strips(int kid, long tn, long Ho, long Wo, long stride) {
    const long room = c3_patch_pixels(kid);
    auto fits = [&](long width) { return largest_patch(tn, width, Ho, stride) <= room; };
    const long widest = (room - 2 * 3 - 3) / 2 / stride + 1;                 // the smallest patch: two rows of the strip and three pixels
    Strips best{0, 0};
    for (long n = ceil_div(Wo, widest); n <= Wo; ++n) {
        const long width = ceil_div(Wo, n), rest = Wo - (ceil_div(Wo, width) - 1) * width;
        if (ceil_div(Wo, width) != n) continue;                               // the same width as with fewer strips
        if (!fits(width) || !fits(rest)) continue;
        const long runs = (n - 1) * ceil_div(width * Ho, tn) + ceil_div(rest * Ho, tn);
        if (best.width == 0 || runs * 33 < best.runs * 32) best = Strips{width, runs};
    }
    return best;
}
// whole blocks of 16 channels; activations and packed weights (three 16-bit parts) within the reach of a buffer descriptor
bool patch_reaches(const Shape& in, const Shape& out) {
    return in.c % 16 == 0 && in.n * in.c * in.h * in.w * 4 < (1L << 31) && 9 * in.c * (out.c + 95) * 6 < (1L << 31);
}
// Which patch kernel a conv3x3 gets (KID_NONE: none fits). Decided from shapes: a compute unit works its workgroups off side by
// side, so the estimate is (tiles per compute unit, rounded up) x a tile's time. One lone workgroup per compute unit cannot keep the
// matrix cores busy on its own: x 1.15, and x 1.25 for 64 x 128 over one or two blocks of channels, mostly filling patches (13 layers of 32
// channels: two rounds of 64 x 64 take 10.6 - 10.9 us there and one of 64 x 128 10.9 - 11.2; with 48 channels 13.2 and 12.6).
// Tiles are the runs of the strips: narrow strips have short runs, which count in full. 128 images of 64 x 33 x 33 to 384 channels,
// stride 2: 64 x 128 with 256 pixels of patch has six runs instead of two and takes 222 us; 64 x 64 takes 119, 64 x 128 with 640 pixels 93.
// The kernels for narrow images take images whose patches hold rows of whole width. Those with 640 pixels take only strides of 2 (at a
// stride of 1 32 x 128 takes 19.8 - 62 us, with 256 pixels 15.3 - 50), 32 x 128 with 256 only strides of 1 (2: 16 images of
// 64 x 45 x 45 -> 32 17.3 us, 64 x 64 with 384 13.1). The others take any width (4 images of 64 channels, stride 1, LDS-staged GEMM / now:
// 159 x 159 -> 32 66 / 30 us, 224 x 224 -> 64 161 / 72, 300 x 300 -> 96 527 / 210; 16 images, stride 2: 90 x 90 -> 64 35 / 25,
// 127 x 127 -> 32 54 / 23, 200 x 200 -> 192 405 / 225).
int choose_patch_kernel(const Shape& in, const Shape& out, long stride, long pad) {
    if (!patch_reaches(in, out)) return KID_NONE;
    int best = KID_NONE;
    double best_cost = 0;
    for (const PatchKernel& k : kPatchKernels) {
        const bool narrow = k.kid == KID_C3_P64 || k.kid == KID_C3_P96;
        if (k.kid == KID_C3_SK || (narrow && patch_pixels(k.tn, in.w, out.h, out.w, stride, pad) > c3_patch_pixels(k.kid))) continue;
        if ((k.tm == 32 && out.c > 32) || (stride == 1 ? c3_patch_pixels(k.kid) == 640 : k.kid == KID_C3_Q32)) continue;
        const Strips strips = choose_strips(k.kid, k.tn, out.h, out.w, stride);
        if (strips.width == 0) continue;
        const long rounds = ceil_div(out.n * strips.runs * ceil_div(out.c, k.tm), 256);
        const double lone = k.tm == 64 && k.tn == 128 && in.c <= 32 ? 1.25 : 1.15;
        const double cost = (double)rounds * k.cost * (rounds == 1 ? lone : 1.0);
        if (best == KID_NONE || cost < best_cost) best = k.kid, best_cost = cost;
    }
    return best;
}
PwChoice choose_c3(const ng_graph* g, int v) {
    PwChoice c;
    const Node& nd = g->nodes[v];
    if (nd.op != NG_OP_CONV3X3) return c;
    const Shape& in = g->nodes[nd.preds[0]].out;
    const long cin = in.c;
    if (cin < 8) return c;
    // The patch-stationary kernels. Few tiles of 64 x 64 (up to two for three compute units) leave the chip idle: 32 x 32 tiles
    // with K over the wavefronts, where the patches are small enough and every wavefront gets a block of 16 channels (with 32
    // channels 5.3 us against 4.1 of the gathering kernel). Us alone, gathering kernel / 64 x 64 tiles / these, tiles of 64 x 64:
    // 17 x 17 192 -> 192 one image 11.5 / 20.9 / 9.2 (15), 14 x 14 192 -> 192 six images 31 / 20 / 10 (72), 35 x 35 96 -> 96
    // four images 34 / 13.4 / 11.3 (160); 30 x 30 64 -> 96 six images 22.6 / 11.0 / 11.8 (180), 8 x 8 384 -> 768 twenty images
    // 196 / 41.5 / 43 (240). Where they don't apply (a stride of 2), from 96 tiles of 64 x 64 on the large tiles: 30 x 30 ->
    // 14 x 14 288 -> 384 six images 80 / 47 (144), one image of 35 x 35 -> 17 x 17 27 / 46 (30). 22 more layers of 64 - 512 channels
    // around the first line, 64 x 64 tiles / these: 120 - 144 tiles 10.3 - 53 / 7.4 - 30.4 (six, these 20 - 45 % faster), 156 - 160
    // 10.6 - 23.9 / 10.6 - 21.5, 180 - 192 10.5 - 52.5 / 10.7 - 40.6, 200 - 250 10.9 - 22.6 / 12.9 - 25.0 (these 9 - 33 % slower). Alone
    // these still win up to three 32 x 32 tiles on a compute unit (27 layers 0.73 - 0.99 of the time, one 1.06); but siblings share launches, which
    // fill the chip with large tiles: with that line the Inception-style network on six images takes 1058 us instead of 1026. 14 more
    // with a stride of 2 around the second, gathering kernel / 64 x 64: 48 tiles 35 / 44.5, 60 - 96 within 7 % of each other, 108
    // 26 / 18 and 67 / 47.5.
    if (!knob("NG_NO_PATCH_KERNELS")) {
        const long tiles64 = nd.out.n * ceil_div(nd.out.h * nd.out.w, 64) * ceil_div(nd.out.c, 64);
        int kid = choose_patch_kernel(in, nd.out, nd.p.stride, nd.p.pad);
        if (patch_reaches(in, nd.out) && cin >= 64 && tiles64 <= 170 && patch_pixels(32, in.w, nd.out.h, nd.out.w, nd.p.stride, nd.p.pad) <= c3_patch_pixels(KID_C3_SK))
            kid = KID_C3_SK;
        else if (nd.out.n * nd.out.h * nd.out.w < kC3LdsMinCols && (cin < 64 || tiles64 < 96))
            kid = KID_NONE;
        for (const PatchKernel& k : kPatchKernels)
            if (k.kid == kid) {
                c.kind = PwChoice::C3_PATCH, c.kid = kid;
                c.groups = (int)cin;                                                             // CinP = Cin (a multiple of 16)
                c.packed = (size_t)(9 * cin) * (size_t)(ceil_div(nd.out.c, k.tm) * k.tm) * 3 / 2;    // [9 Cin / 16][CoutP / 32][3 parts][64 lanes][8 bf16]
                return c;
            }
    }
    if (nd.out.n * nd.out.h * nd.out.w >= kC3LdsMinCols) {
        c.kind = PwChoice::C3_LDS;
        const long kc = nd.out.c <= 32 ? 16 : 32, tm = nd.out.c <= 32 ? 32 : 64;     // K slice and rows per tile of the two kernels
        c.groups = (int)((cin + kc - 1) / kc * kc);                                    // CinP
        c.packed = (size_t)(9 * c.groups) * (size_t)((nd.out.c + tm - 1) / tm * tm);  // W'^T[9 CinP][CoutP]
        return c;
    }
    c.kind = PwChoice::K4_WORD;
    k4_split(9 * cin, nd.out.c, c);
    return c;
}

}  // namespace

// Floats of library-owned constant memory node v needs (repacked conv1x1 weights), 0 if none.
namespace {
// K split of a weight-gradient GEMM: enough workgroups to occupy the GPU, splits of whole K slices
void gemm_split(long m, long n, long k, int* splits, int* k_per_split) {
    const long tiles = ceil_div(m, kGemmTile) * ceil_div(n, kGemmTile);
    // A split costs its share of the K slices (about 0.5 us each) and adds one partial tile to what the workgroup
    // that arrives last has to add up (about 0.4 us each): the sum is smallest near sqrt(1.25 x slices) splits.
    const double slices = (double)ceil_div(k, 16);
    long want = (long)std::lround(std::sqrt(1.25 * slices));
    want = std::max<long>(1, std::min<long>(want, std::max<long>(1, 768 / tiles)));
    const long per = ceil_div(ceil_div(k, want), 16) * 16;
    *k_per_split = (int)per;
    *splits = (int)ceil_div(k, per);
}
// geometry of a weight-gradient node: (M, N, K) of dW[M x N] = dY[M x K] * P^T[K x N]
bool wgrad_dims(const ng_graph* g, int v, long* m, long* n, long* k) {
    const Node& nd = g->nodes[v];
    if (nd.op != NG_OP_CONV1X1_WGRAD && nd.op != NG_OP_CONV3X3_WGRAD) return false;
    const Shape& dy = g->nodes[nd.preds[0]].out;
    const Shape& x = g->nodes[nd.preds[1]].out;
    *m = dy.c, *n = x.c * (nd.op == NG_OP_CONV3X3_WGRAD ? 9 : 1), *k = dy.n * dy.h * dy.w;
    return true;
}
// Workgroups a channel of a batch-norm or depthwise parameter gradient is split over (by images): about 512 workgroups in all
long bn_wgrad_chunks(long channels, long images, long workgroups = 512) {
    const long want = std::max<long>(1, std::min<long>(images, ceil_div(workgroups, channels)));
    return ceil_div(images, ceil_div(images, want));            // no empty chunk
}
long dw_wgrad_chunks(long channels, long images) { return bn_wgrad_chunks(channels, images, knob_int("NG_DW_WGRAD_WGS", 1, 4096, 512)); }
// How a weight-gradient node is computed: which kernel, how K is split, what workspace it needs.
struct WgradPlan {
    bool px = false;              // conv1x1_wgrad_px (both operands 128 bits along the pixels) instead of the gather GEMM
    bool small = false;           // small_gemm: 1 x 1 maps and a few thousand weights (the classifier), no split, no workspace
    int block = 0;                // px: fragments of 16 x 16 weights along each side of a workgroup's block (1 or 2)
    long tiles = 0;
    int splits = 1, k_per_split = 0;
    size_t ws_floats = 0;         // partial tiles (and group sums)
    size_t cnt_words = 0;         // arrival counters behind them, a multiple of 64
};
WgradPlan wgrad_plan(const ng_graph* g, int v) {
    WgradPlan p;
    long m, n, k;
    if (!wgrad_dims(g, v, &m, &n, &k)) return p;
    const Node& nd = g->nodes[v];
    const Shape& dy = g->nodes[nd.preds[0]].out;
    const Shape& x = g->nodes[nd.preds[1]].out;
    p.tiles = ceil_div(m, kGemmTile) * ceil_div(n, kGemmTile);
    const size_t tile_floats = (size_t)kGemmTile * kGemmTile;
    if (nd.op == NG_OP_CONV1X1_WGRAD && dy.h * dy.w == 1 && m * n <= kSmallGemmOutputs && k <= kSmallGemmK) {
        p.small = true, p.splits = 1, p.k_per_split = (int)k;
        return p;
    }
    const long hw = dy.h * dy.w;
    const bool c3 = nd.op == NG_OP_CONV3X3_WGRAD, whole = c3 ? dy.w % 16 == 0 : hw % 16 == 0;
    p.px = hw >= 4 && (whole || k >= kRaggedMinPixels) && dy.elems() * 4 < (1L << 31) && x.elems() * 4 < (1L << 31) &&
           (!c3 || (nd.p.stride == 1 && nd.p.pad == 1 && dy.w >= 4 && dy.h == x.h && dy.w == x.w));
    k = dy.n * ceil_div(hw, 16) * 16;                           // an image is a whole number of slices of 16 pixels
    const long fm = ceil_div(m, 16), fn = ceil_div(n, 16);
    p.px = p.px && fm * fn <= 256;
    if (p.px) {
        // Blocks of B x B fragments of 16 x 16 weights, each split over K: 512 pixels a split (eight slices of 16 for each of
        // the four wavefronts: one batch of loads) up to 128 splits, which somebody has to add up; where that leaves compute
        // units idle, 256 pixels for about two workgroups each. Training step of a NAS cell with 44 channels on 32 x 32
        // maps: batch 32 (64 splits) 1072 us, with 128 splits 1097; batch 96 (128 splits) 2187 us, with 64 splits 2220 -
        // 2230, with 32 splits 2266.
        p.block = fm * fn <= 16 ? 1 : 2;
        p.tiles = ceil_div(fm, p.block) * ceil_div(fn, p.block);
        const long most = 128;
        const long want = std::max<long>({1, std::min(k / 512, most), std::min<long>({ceil_div(k, 256), 512 / p.tiles, 64})});
        // of the splits near that (each a multiple of 64 pixels) the one whose XCDs, which take every eighth split, are
        // busiest for the shortest time
        long best = -1;
        for (long per = ceil_div(ceil_div(k, std::min(want * 5 / 4, most)), 64); per <= ceil_div(ceil_div(k, std::max<long>(1, want * 3 / 4)), 64); ++per) {
            const long cost = ceil_div(ceil_div(k, per * 64), 8) * per;
            if (best < 0 || cost < best) best = cost, p.k_per_split = (int)(per * 64);
        }
        p.splits = (int)ceil_div(k, p.k_per_split);
        if (p.splits > 1) {
            p.ws_floats = (size_t)p.tiles * p.splits * 256 * p.block * p.block;
            p.cnt_words = ((size_t)p.tiles + 63) & ~(size_t)63;
        }
        return p;
    }
    gemm_split(m, n, dy.n * hw, &p.splits, &p.k_per_split);
    if (p.splits > 1) {
        p.ws_floats = (size_t)p.tiles * p.splits * tile_floats;
        p.cnt_words = ((size_t)p.tiles + 63) & ~(size_t)63;
    }
    return p;
}
}  // namespace

size_t packed_floats(const ng_graph* g, int v) {
    const Node& nd = g->nodes[v];
    long wm, wn, wk;
    if (wgrad_dims(g, v, &wm, &wn, &wk)) {                     // split-K workspace: partial tiles, then the arrival counters
        const WgradPlan p = wgrad_plan(g, v);
        return p.ws_floats + p.cnt_words;
    }
    if (nd.op == NG_OP_DWCONV_WGRAD) {                         // per-chunk partial sums [C][chunks][K K] (padded), then one arrival counter per channel
        const Shape& x = g->nodes[nd.preds[1]].out;
        const long chunks = dw_wgrad_chunks(x.c, x.n);
        return chunks > 1 ? (size_t)((x.c * chunks * nd.p.k * nd.p.k + 63) & ~63L) + (size_t)((x.c + 63) & ~63L) : 0;
    }
    if (nd.op == NG_OP_BN_ACT_WGRAD) {                         // per-chunk sums [C][chunks][2] (padded), then one arrival counter per channel
        const Shape& x = g->nodes[nd.preds[1]].out;
        const long chunks = bn_wgrad_chunks(x.c, x.n);
        return chunks > 1 ? (size_t)((x.c * chunks * 2 + 63) & ~63L) + (size_t)((x.c + 63) & ~63L) : 0;
    }
    if (g->trainable) return 0;                                // weights change between replays: nothing is folded or repacked
    if (nd.op == NG_OP_BN_ACT) return 2 * (size_t)((nd.out.c + 3) & ~3L);   // folded scale, shift
    if (nd.op == NG_OP_CONV3X3) return choose_c3(g, v).packed;
    return choose_pw(g, v).packed;
}

// Fill node v's constant memory: one pass over the weights, at bind time.
int pack_constants(ng_graph* g, int v, float* packed, void* stream) {
    const Node& nd = g->nodes[v];
    long wm, wn, wk;
    if (wgrad_dims(g, v, &wm, &wn, &wk)) {                     // the arrival counters start at zero
        const WgradPlan p = wgrad_plan(g, v);
        if (p.cnt_words == 0) return NG_OK;
        const hipError_t e = hipMemsetAsync(packed + p.ws_floats, 0, p.cnt_words * sizeof(float), static_cast<hipStream_t>(stream));
        if (e != hipSuccess) return g->fail(NG_EHIP, "clearing split-K counters: %s", hipGetErrorString(e));
        return NG_OK;
    }
    if (nd.op == NG_OP_DWCONV_WGRAD || nd.op == NG_OP_BN_ACT_WGRAD) {
        const size_t floats = packed_floats(g, v);
        if (floats == 0) return NG_OK;
        const size_t cnt = (size_t)((g->nodes[nd.preds[1]].out.c + 63) & ~63L);
        const hipError_t e = hipMemsetAsync(packed + floats - cnt, 0, cnt * sizeof(float), static_cast<hipStream_t>(stream));
        if (e != hipSuccess) return g->fail(NG_EHIP, "clearing depthwise wgrad counters: %s", hipGetErrorString(e));
        return NG_OK;
    }
    if (g->trainable) return NG_OK;
    if (nd.op == NG_OP_BN_ACT) {
        for (int j = 0; j < 4; ++j)
            if (!nd.weights[j]) return g->fail(NG_EINVAL, "node %d: weight %d is a null device pointer", v, j);
        const int C = (int)nd.out.c;
        fold_bn_kernel<<<dim3((unsigned)((C + kBlock - 1) / kBlock)), dim3(kBlock), 0, static_cast<hipStream_t>(stream)>>>(
            static_cast<const float*>(nd.weights[0]), static_cast<const float*>(nd.weights[1]),
            static_cast<const float*>(nd.weights[2]), static_cast<const float*>(nd.weights[3]), nd.p.eps, packed,
            packed + ((C + 3) & ~3), C);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return g->fail(NG_EHIP, "folding batch-norm parameters: %s", hipGetErrorString(e));
        return NG_OK;
    }
    const bool c3 = nd.op == NG_OP_CONV3X3;
    const PwChoice c = c3 ? choose_c3(g, v) : choose_pw(g, v);
    if (c.packed == 0) return NG_OK;
    const int cin = (int)g->nodes[nd.preds[0]].out.c * (c3 ? 9 : 1), cout = (int)nd.out.c;
    if (!nd.weights[0]) return g->fail(NG_EINVAL, "node %d: weight 0 is a null device pointer", v);
    const dim3 grid((unsigned)((c.packed + kBlock - 1) / kBlock)), block(kBlock);
    if (c.kind == PwChoice::PW_PATCH || c.kind == PwChoice::C3_PATCH) {
        const long threads = (long)(c.packed / 12);             // one per 8 weights in three parts of 16 bits
        pack_split_weights_kernel<<<dim3((unsigned)ceil_div(threads, kBlock)), block, 0, static_cast<hipStream_t>(stream)>>>(
            static_cast<const float*>(nd.weights[0]), packed, cout, c.groups, c3 ? 9 : 1,
            (int)(c.packed / ((size_t)cin / 16 * (kSplitFragBytes / 4))), threads);
    }
    else if (c.kind == PwChoice::LDS64)
        pack_pw_lds_weights_kernel<<<grid, block, 0, static_cast<hipStream_t>(stream)>>>(
            static_cast<const float*>(nd.weights[0]), packed, cout, cin, (int)(c.packed / (size_t)c.groups), (long)c.packed);
    else if (c.kind == PwChoice::C3_LDS)
        pack_c3_lds_weights_kernel<<<grid, block, 0, static_cast<hipStream_t>(stream)>>>(
            static_cast<const float*>(nd.weights[0]), packed, cout, cin / 9, c.groups, (int)(c.packed / (9 * (size_t)c.groups)), (long)c.packed);
    else if (c.kind == PwChoice::DIRECT32)
        pack_pw_weights_kernel<<<grid, block, 0, static_cast<hipStream_t>(stream)>>>(
            static_cast<const float*>(nd.weights[0]), packed, cout, cin, c.groups, (int)c.packed);
    else
        pack_pw_weights_k4_kernel<<<grid, block, 0, static_cast<hipStream_t>(stream)>>>(
            static_cast<const float*>(nd.weights[0]), packed, cout, cin, c.groups, (int)c.packed);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return g->fail(NG_EHIP, "repacking conv1x1 weights: %s", hipGetErrorString(e));
    return NG_OK;
}

int build_task(ng_graph* g, int v, char* arena, float* packed, Task& t) {
    const Node& nd = g->nodes[v];
    t = Task();
    t.block[0] = kBlock;
    if (nd.op == NG_OP_INPUT) return NG_OK;
    for (size_t j = 0; j < nd.weights.size(); ++j)
        if (!nd.weights[j] && !g->dry_run) return g->fail(NG_EINVAL, "node %d: weight %d is a null device pointer", v, (int)j);

    auto buf = [&](int id) { return reinterpret_cast<float*>(arena + g->offset[id]); };
    const Shape& o = nd.out;
    const Shape& i0 = g->nodes[nd.preds[0]].out;
    const int total = (int)o.elems();
    const int hw_out = (int)(o.h * o.w);
    auto wf = [&](int j) { return static_cast<const float*>(nd.weights[j]); };

    switch (nd.op) {
        case NG_OP_BN_ACT:
            if (g->trainable) {                                   // gamma and beta change between replays: no folded copy
                BnRawArgs a{};
                a.x = buf(nd.preds[0]), a.y = buf(v);
                a.gamma = wf(0), a.beta = wf(1), a.mean = wf(2), a.var = wf(3);
                a.eps = nd.p.eps, a.relu = nd.p.relu != 0;
                a.C = (int)o.c, a.HW = hw_out, a.N = (int)o.n, a.total = total;
                set_kernel<KID_BN_RAW>(t, a, ceil_div(total, kBlock));
                break;
            }
            [[fallthrough]];
        case NG_OP_RELU: {
            BnArgs a{};
            a.x = buf(nd.preds[0]);
            a.y = buf(v);
            if (nd.op == NG_OP_BN_ACT) {
                if (!packed) return g->fail(NG_EINVAL, "node %d: no buffer for folded batch-norm parameters", v);
                a.scale = packed, a.shift = packed + ((o.c + 3) & ~3L);
                a.relu = nd.p.relu != 0;
            } else {
                a.relu = 1;
            }
            a.C = (int)o.c, a.HW = hw_out, a.total = total;
            a.cols = (int)(o.n * hw_out);
            if (hw_out % 4 == 0) set_kernel<KID_BN_V4>(t, a, ceil_div(total / 4, kBlock));
            else set_kernel<KID_BN>(t, a, ceil_div(total, kBlock));
            break;
        }
        case NG_OP_ADD_N: {
            AddArgs a{};
            a.k = (int)nd.preds.size();
            for (int j = 0; j < NG_MAX_PREDS; ++j) a.x[j] = buf(nd.preds[j < a.k ? j : 0]);
            a.y = buf(v);
            a.total = total;
            a.C = (int)o.c, a.HW = hw_out, a.cols = (int)(o.n * hw_out);
            if (total % 4 == 0) set_kernel<KID_ADD_V4>(t, a, ceil_div(total / 4, kBlock));
            else set_kernel<KID_ADD>(t, a, ceil_div(total, kBlock));
            break;
        }
        case NG_OP_CONCAT: {
            ConcatArgs a{};
            a.k = (int)nd.preds.size();
            int first = 0;
            for (int j = 0; j < a.k; ++j) {
                a.x[j] = buf(nd.preds[j]);
                a.cin[j] = (int)g->nodes[nd.preds[j]].out.c;
                a.lo[j] = nd.p.slice_lo[j];
                a.first[j] = first;
                first += nd.p.slice_hi[j] - nd.p.slice_lo[j];
            }
            for (int j = a.k; j < NG_MAX_PREDS; ++j) a.x[j] = a.x[0], a.first[j] = first;
            a.y = buf(v);
            a.C = (int)o.c, a.HW = hw_out, a.total = total;
            // 128 bits at a time wherever four elements never straddle two blocks or two images, on either side: every block
            // starts at and has a multiple of four elements (odd maps with channels in fours as well; an Inception-style
            // network at batch 32, whose concats are of 35 x 35 and 17 x 17 maps, 3666 -> 3571 us)
            bool quads = true;
            for (int j = 0; j < a.k; ++j)
                quads = quads && (long)a.first[j] * hw_out % 4 == 0 && (long)a.lo[j] * hw_out % 4 == 0 && (long)a.cin[j] * hw_out % 4 == 0;
            quads = quads && (long)a.C * hw_out % 4 == 0;
            if (quads) set_kernel<KID_CONCAT_V4>(t, a, ceil_div(total / 4, kBlock));
            else set_kernel<KID_CONCAT>(t, a, ceil_div(total, kBlock));
            break;
        }
        case NG_OP_POOL: {
            PoolArgs a{buf(nd.preds[0]), buf(v), (int)i0.h, (int)i0.w, (int)o.h, (int)o.w,
                       nd.p.stride, nd.p.pad, nd.p.pool_mode, total};
            // large tensors (batches): four outputs of a column per thread
            if (total >= kPoolRowMinOutputs && (nd.p.stride == 1 || nd.p.stride == 2)) {
                const long items = (long)o.n * o.c * ceil_div(o.h, 4) * o.w;
                if (nd.p.stride == 1) set_kernel<KID_POOL_ROW_S1>(t, a, ceil_div(items, kBlock));
                else set_kernel<KID_POOL_ROW_S2>(t, a, ceil_div(items, kBlock));
                break;
            }
            set_kernel<KID_POOL>(t, a, ceil_div(total, kBlock));
            break;
        }
        case NG_OP_DWCONV: {
            DwArgs a{buf(nd.preds[0]), wf(0), buf(v), (int)o.c, (int)i0.h, (int)i0.w, (int)o.h, (int)o.w, total};
            const long n = ceil_div(total, kBlock);
            // large tensors of small planes (batches): whole planes through LDS, four outputs per thread
            const long quads = i0.h * ceil_div(i0.w, 4), per_wg = planes_in_lds((int)i0.h, (int)i0.w, nd.p.k);
            if (total >= kDwLdsMinOutputs && (nd.p.k == 3 || nd.p.k == 5) && (nd.p.stride == 1 || nd.p.stride == 2) && i0.w >= 4 &&
                o.w >= 4 && per_wg > 0 && o.h * ceil_div(o.w, 4) <= quads) {
                a.K = nd.p.k, a.S = nd.p.stride, a.planes_per_tile = (int)per_wg;
                set_kernel<KID_DW_LDS>(t, a, ceil_div((long)o.n * o.c, per_wg));
                break;
            }
            if (nd.p.k == 3 && nd.p.stride == 1) set_kernel<KID_DW_K3S1>(t, a, n);
            else if (nd.p.k == 3) set_kernel<KID_DW_K3S2>(t, a, n);
            else if (nd.p.stride == 1) set_kernel<KID_DW_K5S1>(t, a, n);
            else set_kernel<KID_DW_K5S2>(t, a, n);
            break;
        }
        case NG_OP_GLOBAL_AVGPOOL: {
            GapArgs a{buf(nd.preds[0]), buf(v), (int)(i0.h * i0.w), (int)(o.n * o.c)};
            set_kernel<KID_GAP>(t, a, ceil_div(a.planes, kBlock / 64));
            break;
        }
        case NG_OP_FC:
        case NG_OP_CONV1X1: {
            const bool fc = nd.op == NG_OP_FC;
            if (g->trainable) {                                   // weights change between replays: read them where they are
                GemmArgs a{};
                a.a = wf(0), a.b = buf(nd.preds[0]), a.c = buf(v), a.bias = fc ? wf(1) : nullptr;
                a.M = (int)o.c, a.K = (int)i0.c, a.N = (int)(o.n * hw_out);
                a.Cin = (int)i0.c, a.Cout = (int)o.c, a.H = a.Ho = (int)o.h, a.W = a.Wo = (int)o.w, a.stride = 1;
                a.tiles_n = (int)ceil_div(a.N, kGemmTile), a.splits = 1, a.k_per_split = a.K;
                if (hw_out == 1 && (long)a.M * a.N <= kSmallGemmOutputs && a.K <= kSmallGemmK) {
                    // Y[n][o] = sum_k W[o][k] X[n][k] + b[o]
                    SmallGemmArgs sg{a.a, a.b, a.c, a.bias, a.M, a.N, a.K, a.K, 1, 1, a.K, 1, a.M, 0};
                    set_small_gemm(t, sg, [](Task& tt, const SmallGemmArgs& aa, long n) { set_kernel<KID_SMALL_GEMM>(tt, aa, n); });
                    break;
                }
                if (!fc && pw_px_applies(a)) set_kernel<KID_PW_PX_FWD>(t, a, pw_px_tiles(a));
                else set_kernel<KID_GEMM_PW_FWD>(t, a, (long)a.tiles_n * ceil_div(a.M, kGemmTile));
                break;
            }
            const PwChoice c = choose_pw(g, v);
            if (c.kind == PwChoice::GEMV) {
                FcArgs a{buf(nd.preds[0]), wf(0), wf(1), buf(v), (int)o.n, (int)i0.c, (int)o.c};
                set_kernel<KID_FC_GEMV>(t, a, ceil_div(a.Cout, kBlock / 64));
                break;
            }
            PwArgs a{};
            a.x = buf(nd.preds[0]), a.w = wf(0), a.bias = fc ? wf(1) : nullptr, a.y = buf(v);
            a.Cin = (int)i0.c, a.Cout = (int)o.c, a.HW = hw_out, a.cols = (int)(o.n * hw_out);
            if (c.kind == PwChoice::PW_PATCH) {
                if (!packed) return g->fail(NG_EINVAL, "node %d: no buffer for repacked weights", v);
                a.wp = packed, a.ksteps = c.groups;
                a.tiles_n = (int)ceil_div(a.cols, 64);
                a.mtiles = (int)ceil_div(a.Cout, c.kid == KID_PW_P32 ? 32 : 64);
                if (c.kid == KID_PW_P32) set_kernel<KID_PW_P32>(t, a, (long)a.tiles_n * a.mtiles);
                else set_kernel<KID_PW_P64>(t, a, (long)a.tiles_n * a.mtiles);
                break;
            }
            if (c.kind == PwChoice::LDS64) {
                if (!packed) return g->fail(NG_EINVAL, "node %d: no buffer for repacked weights", v);
                a.wp = packed, a.ksteps = c.groups;
                a.tiles_n = (int)ceil_div(a.cols, 64);
                set_kernel<KID_PW_64>(t, a, (long)a.tiles_n * ceil_div(a.Cout, 64));
                break;
            }
            if (!packed) return g->fail(NG_EINVAL, "node %d: no buffer for repacked weights", v);
            a.wp = packed;
            a.ksteps = c.groups;
            a.mtiles = (int)ceil_div(a.Cout, 16);
            if (c.kind == PwChoice::DIRECT32) {
                a.tiles_n = (int)ceil_div(a.cols, 32);
                const long n = (long)a.tiles_n * ceil_div(a.Cout, 32);
                if (c.in_flight == 4) set_kernel<KID_PW_D4>(t, a, n);
                else if (c.in_flight == 8) set_kernel<KID_PW_D8>(t, a, n);
                else set_kernel<KID_PW_D16>(t, a, n);
            } else if (c.kind == PwChoice::K4_VEC) {
                a.tiles_n = (int)ceil_div(a.cols, 64);
                const long n = (long)a.tiles_n * a.mtiles;
                if (c.in_flight == 1) set_kernel<KID_PW_V1>(t, a, n);
                else if (c.in_flight == 2) set_kernel<KID_PW_V2>(t, a, n);
                else if (c.in_flight == 3) set_kernel<KID_PW_V3>(t, a, n);
                else set_kernel<KID_PW_V4>(t, a, n);
            } else {
                a.tiles_n = (int)ceil_div(a.cols, 16);
                const long n = (long)a.tiles_n * a.mtiles;
                if (c.in_flight == 1) set_kernel<KID_PW_S1>(t, a, n);
                else if (c.in_flight == 2) set_kernel<KID_PW_S2>(t, a, n);
                else if (c.in_flight == 3) set_kernel<KID_PW_S3>(t, a, n);
                else set_kernel<KID_PW_S4>(t, a, n);
            }
            break;
        }
        case NG_OP_CONV3X3: {
            C3Args a{};
            a.x = buf(nd.preds[0]), a.w = wf(0), a.y = buf(v);
            a.Cin = (int)i0.c, a.Cout = (int)o.c, a.H = (int)i0.h, a.W = (int)i0.w, a.Ho = (int)o.h, a.Wo = (int)o.w;
            a.pad = nd.p.pad, a.stride = nd.p.stride;
            if (g->trainable) {
                GemmArgs ga{};
                ga.a = wf(0), ga.b = buf(nd.preds[0]), ga.c = buf(v);
                ga.M = (int)o.c, ga.K = (int)i0.c * 9, ga.N = (int)(o.n * o.h * o.w);
                ga.Cin = (int)i0.c, ga.Cout = (int)o.c, ga.H = (int)i0.h, ga.W = (int)i0.w, ga.Ho = (int)o.h, ga.Wo = (int)o.w;
                ga.stride = nd.p.stride, ga.pad = nd.p.pad;
                ga.tiles_n = (int)ceil_div(ga.N, kGemmTile), ga.splits = 1, ga.k_per_split = ga.K;
                set_kernel<KID_GEMM_C3_FWD>(t, ga, (long)ga.tiles_n * ceil_div(ga.M, kGemmTile));
                break;
            }
            const PwChoice c = choose_c3(g, v);
            if (c.kind == PwChoice::C3_PATCH) {
                if (!packed) return g->fail(NG_EINVAL, "node %d: no buffer for repacked weights", v);
                a.wp = packed, a.groups = c.groups;
                a.cols = (int)(o.n * o.h * o.w);
                for (const PatchKernel& k : kPatchKernels) {
                    if (k.kid != c.kid) continue;
                    // runs of pixels per image; conv3x3_mfma_split_k takes rows of whole width
                    const Strips strips = k.kid == KID_C3_SK ? Strips{o.w, ceil_div(o.h * o.w, k.tn)} : choose_strips(k.kid, k.tn, o.h, o.w, nd.p.stride);
                    a.tiles_x = (int)strips.width, a.tiles_xy = (int)strips.runs;
                    a.tiles_n = (int)o.n * a.tiles_xy;
                    a.co_groups = (int)ceil_div(a.Cout, k.tm);
                }
                const long n = (long)a.tiles_n * a.co_groups;
                switch (c.kid) {
                    case KID_C3_P64: set_kernel<KID_C3_P64>(t, a, n); break;
                    case KID_C3_P96: set_kernel<KID_C3_P96>(t, a, n); break;
                    case KID_C3_Q32: set_kernel<KID_C3_Q32>(t, a, n); break;
                    case KID_C3_Q64: set_kernel<KID_C3_Q64>(t, a, n); break;
                    case KID_C3_R32: set_kernel<KID_C3_R32>(t, a, n); break;
                    case KID_C3_R128: set_kernel<KID_C3_R128>(t, a, n); break;
                    case KID_C3_SK: set_kernel<KID_C3_SK>(t, a, n); break;
                    default: set_kernel<KID_C3_Q128>(t, a, n); break;
                }
                break;
            }
            if (c.kind == PwChoice::C3_LDS) {
                if (!packed) return g->fail(NG_EINVAL, "node %d: no buffer for repacked weights", v);
                a.wp = packed, a.groups = c.groups;
                a.cols = (int)(o.n * o.h * o.w);
                if (a.Cout <= 32) {
                    a.tiles_n = (int)ceil_div(a.cols, 128);
                    set_kernel<KID_C3_L32>(t, a, (long)a.tiles_n * ceil_div(a.Cout, 32));
                } else {
                    a.tiles_n = (int)ceil_div(a.cols, 64);
                    set_kernel<KID_C3_L64>(t, a, (long)a.tiles_n * ceil_div(a.Cout, 64));
                }
                break;
            }
            if (c.packed != 0) {
                if (!packed) return g->fail(NG_EINVAL, "node %d: no buffer for repacked weights", v);
                a.wp = packed, a.groups = c.groups;
                a.cols = (int)(o.n * o.h * o.w), a.tiles_n = (int)ceil_div(a.cols, 16);
                const long n = (long)a.tiles_n * ceil_div(a.Cout, 16);
                if (c.in_flight == 1) set_kernel<KID_C3_M1>(t, a, n);
                else if (c.in_flight == 2) set_kernel<KID_C3_M2>(t, a, n);
                else if (c.in_flight == 3) set_kernel<KID_C3_M3>(t, a, n);
                else set_kernel<KID_C3_M4>(t, a, n);
                break;
            }
            // small maps: 8 x 8 tiles waste fewer lanes; a stem at batch 1 (3 input channels, a large map): four times the
            // workgroups, each with a quarter of the patch to load
            const bool small = o.h * o.w <= 24 * 24 || (a.Cin <= 4 && o.n == 1);
            const int tp = small ? 8 : 16;
            a.tiles_x = (int)ceil_div(o.w, tp);
            a.tiles_xy = a.tiles_x * (int)ceil_div(o.h, tp);
            a.co_groups = (int)ceil_div(a.Cout, small ? 32 : 8);
            const long n = (long)a.tiles_xy * a.co_groups * o.n;
            if (small) {
                if (nd.p.stride == 1) set_kernel<KID_C3_T8S1>(t, a, n); else set_kernel<KID_C3_T8S2>(t, a, n);
            } else {
                if (nd.p.stride == 1) set_kernel<KID_C3_T16S1>(t, a, n); else set_kernel<KID_C3_T16S2>(t, a, n);
            }
            break;
        }
        // ---- backward operators and the weight update (graphs that train) ----
        case NG_OP_CONV1X1_DGRAD:
        case NG_OP_CONV3X3_DGRAD: {
            const bool c3 = nd.op == NG_OP_CONV3X3_DGRAD;
            const Shape& dy = i0;                                 // [n][Cout][Ho][Wo]; the result has the shape of the forward input
            GemmArgs a{};
            a.a = wf(0), a.b = buf(nd.preds[0]), a.c = buf(v);
            a.Cin = (int)o.c, a.Cout = (int)dy.c, a.H = (int)o.h, a.W = (int)o.w, a.Ho = (int)dy.h, a.Wo = (int)dy.w;
            a.stride = c3 ? nd.p.stride : 1, a.pad = c3 ? nd.p.pad : 0;
            a.M = a.Cin, a.K = a.Cout * (c3 ? 9 : 1), a.N = (int)(o.n * o.h * o.w);
            a.tiles_n = (int)ceil_div(a.N, kGemmTile), a.splits = 1, a.k_per_split = a.K;
            const long n = (long)a.tiles_n * ceil_div(a.M, kGemmTile);
            if (!c3 && o.h * o.w == 1 && (long)a.M * a.N <= kSmallGemmOutputs && a.K <= kSmallGemmK) {
                // dX[n][ci] = sum_co W[co][ci] dY[n][co]
                SmallGemmArgs sg{a.a, a.b, a.c, nullptr, a.M, a.N, a.K, 1, a.M, 1, a.K, 1, a.M, 0};
                set_small_gemm(t, sg, [](Task& tt, const SmallGemmArgs& aa, long n2) { set_kernel<KID_SMALL_GEMM>(tt, aa, n2); });
                break;
            }
            if (c3) set_kernel<KID_GEMM_C3_DGRAD>(t, a, n);
            else if (pw_px_applies(a)) set_kernel<KID_PW_PX_DGRAD>(t, a, pw_px_tiles(a));
            else set_kernel<KID_GEMM_PW_DGRAD>(t, a, n);
            break;
        }
        case NG_OP_CONV1X1_WGRAD:
        case NG_OP_CONV3X3_WGRAD: {
            const bool c3 = nd.op == NG_OP_CONV3X3_WGRAD;
            const Shape& dy = i0;
            const Shape& x = g->nodes[nd.preds[1]].out;
            GemmArgs a{};
            a.a = buf(nd.preds[0]), a.b = buf(nd.preds[1]), a.c = buf(v);
            a.Cin = (int)x.c, a.Cout = (int)dy.c, a.H = (int)x.h, a.W = (int)x.w, a.Ho = (int)dy.h, a.Wo = (int)dy.w;
            a.stride = c3 ? nd.p.stride : 1, a.pad = c3 ? nd.p.pad : 0;
            a.M = a.Cout, a.N = a.Cin * (c3 ? 9 : 1), a.K = (int)(dy.n * dy.h * dy.w);
            a.tiles_n = (int)ceil_div(a.N, kGemmTile);
            const WgradPlan p = wgrad_plan(g, v);
            a.splits = p.splits, a.k_per_split = p.k_per_split;
            const long tiles = p.tiles;
            if (a.splits > 1) {
                if (!packed) return g->fail(NG_EINVAL, "node %d: no workspace for the split-K partial tiles", v);
                a.ws = packed;
                a.cnt = reinterpret_cast<unsigned*>(packed + p.ws_floats);
            }
            if (p.small) {
                // dW[co][ci] = sum_n dY[n][co] X[n][ci]
                SmallGemmArgs sg{a.a, a.b, a.c, nullptr, a.M, a.N, a.K, 1, a.M, a.N, 1, a.N, 1, 0};
                set_small_gemm(t, sg, [](Task& tt, const SmallGemmArgs& aa, long n2) { set_kernel<KID_SMALL_GEMM>(tt, aa, n2); });
                break;
            }
            if (p.px) a.tiles_n = (int)ceil_div(ceil_div(a.N, 16), p.block);
            if (p.px && c3 && p.block == 1) set_kernel<KID_C3_WGRAD_PX>(t, a, tiles * a.splits);
            else if (p.px && c3) set_kernel<KID_C3_WGRAD_PX2>(t, a, tiles * a.splits);
            else if (p.px && p.block == 1) set_kernel<KID_PW_WGRAD_PX>(t, a, tiles * a.splits);
            else if (p.px) set_kernel<KID_PW_WGRAD_PX2>(t, a, tiles * a.splits);
            else if (c3) set_kernel<KID_GEMM_C3_WGRAD>(t, a, tiles * a.splits);
            else set_kernel<KID_GEMM_PW_WGRAD>(t, a, tiles * a.splits);
            break;
        }
        case NG_OP_BN_ACT_DGRAD:
        case NG_OP_BN_ACT_WGRAD: {
            const Shape& x = g->nodes[nd.preds[1]].out;
            BnRawArgs a{};
            a.dy = buf(nd.preds[0]), a.x = buf(nd.preds[1]), a.y = buf(v);
            a.gamma = wf(0), a.beta = wf(1), a.mean = wf(2), a.var = wf(3);
            a.eps = nd.p.eps, a.relu = nd.p.relu != 0;
            a.C = (int)x.c, a.HW = (int)(x.h * x.w), a.N = (int)x.n, a.total = (int)x.elems();
            if (nd.op == NG_OP_BN_ACT_DGRAD) {
                set_kernel<KID_BN_DGRAD>(t, a, ceil_div(a.total, kBlock));
                break;
            }
            a.chunks = (int)bn_wgrad_chunks(a.C, a.N);
            if (a.chunks > 1) {
                if (!packed) return g->fail(NG_EINVAL, "node %d: no workspace for the per-chunk sums", v);
                a.ws = packed;
                a.cnt = reinterpret_cast<unsigned*>(packed + (((size_t)a.C * a.chunks * 2 + 63) & ~(size_t)63));
            }
            set_kernel<KID_BN_WGRAD>(t, a, (long)a.C * a.chunks);
            break;
        }
        case NG_OP_RELU_DGRAD:
        case NG_OP_GAP_DGRAD:
        case NG_OP_SLICE_PAD:
        case NG_OP_CHANNEL_SUM: {
            EltGradArgs a{};
            a.dy = buf(nd.preds[0]), a.x = nd.preds.size() > 1 ? buf(nd.preds[1]) : nullptr, a.y = buf(v);
            a.C = (int)o.c, a.HW = hw_out, a.N = (int)o.n, a.total = total;
            if (nd.op == NG_OP_RELU_DGRAD) {
                set_kernel<KID_RELU_DGRAD>(t, a, ceil_div(total, kBlock));
            } else if (nd.op == NG_OP_GAP_DGRAD) {
                a.scale = 1.f / (float)hw_out;
                set_kernel<KID_GAP_DGRAD>(t, a, ceil_div(total, kBlock));
            } else if (nd.op == NG_OP_SLICE_PAD) {
                a.src_C = (int)i0.c, a.src_lo = nd.p.slice_lo[0], a.cnt = nd.p.slice_hi[0] - nd.p.slice_lo[0], a.dst_lo = nd.p.slice_lo[1];
                set_kernel<KID_SLICE_PAD>(t, a, ceil_div(total, kBlock));
            } else {                                              // sums run over the input's images and pixels
                a.C = (int)i0.c, a.HW = (int)(i0.h * i0.w), a.N = (int)i0.n;
                set_kernel<KID_CHANNEL_SUM>(t, a, a.C);
            }
            break;
        }
        case NG_OP_DWCONV_DGRAD:
        case NG_OP_DWCONV_WGRAD: {
            const Shape& dy = i0;
            const Shape& x = g->nodes[nd.preds[1]].out;
            DwGradArgs a{};
            a.dy = buf(nd.preds[0]), a.x = buf(nd.preds[1]), a.y = buf(v);
            a.N = (int)x.n, a.C = (int)x.c, a.H = (int)x.h, a.W = (int)x.w, a.Ho = (int)dy.h, a.Wo = (int)dy.w;
            a.K = nd.p.k, a.S = nd.p.stride, a.total = (int)x.elems();
            if (nd.op == NG_OP_DWCONV_DGRAD) {
                a.w = wf(0);
                const long plane = (long)a.H * a.W, planes = a.total / plane;
                const long quads = a.H * ceil_div(a.W, 4);
                // planes of dx of at most 256 quads; their dy planes, which are no larger, in LDS
                const long per_wg = quads <= kBlock ? std::min<long>(kBlock / quads, (kSmemFloats - kPlaneSlack) / plane_floats(a.Ho, a.Wo, a.K)) : 0;
                const bool whole = a.W % 4 == 0 && a.Wo % 4 == 0;
                if ((a.K == 3 || a.K == 5) && (a.S == 1 || a.S == 2) && a.W >= 4 && a.Wo >= 4 && per_wg > 0 &&
                    a.Ho * ceil_div(a.Wo, 4) <= quads && (whole || a.total >= kRaggedMinElements)) {
                    a.chunks = (int)per_wg;                        // whole planes of dx per workgroup, their dy staged in LDS
                    set_kernel<KID_DW_DGRAD_LDS>(t, a, ceil_div(planes, per_wg));
                    break;
                }
                set_kernel<KID_DW_DGRAD>(t, a, ceil_div(a.total, kBlock));
            } else {
                a.chunks = (int)dw_wgrad_chunks(a.C, a.N);
                if (a.chunks > 1) {
                    if (!packed) return g->fail(NG_EINVAL, "node %d: no workspace for the per-chunk partial sums", v);
                    a.ws = packed;
                    a.cnt = reinterpret_cast<unsigned*>(packed + (((size_t)a.C * a.chunks * a.K * a.K + 63) & ~(size_t)63));
                }
                set_kernel<KID_DW_WGRAD>(t, a, (long)a.C * a.chunks);
            }
            break;
        }
        case NG_OP_POOL_DGRAD: {
            const Shape& dy = i0;
            const Shape& x = g->nodes[nd.preds[1]].out;
            PoolGradArgs a{buf(nd.preds[0]), buf(nd.preds[1]), buf(v), (int)x.h, (int)x.w, (int)dy.h, (int)dy.w,
                           nd.p.stride, nd.p.pad, nd.p.pool_mode, (int)x.elems()};
            const long plane = (long)x.h * x.w;
            if (plane <= kPoolGradChunk && dy.h * dy.w <= plane) {      // whole planes fit a workgroup's LDS
                a.planes_per_tile = (int)(kPoolGradChunk / plane);
                set_kernel<KID_POOL_DGRAD_LDS>(t, a, ceil_div(a.total / plane, a.planes_per_tile));
            } else {
                set_kernel<KID_POOL_DGRAD>(t, a, ceil_div(a.total, kBlock));
            }
            break;
        }
        case NG_OP_SGD_UPDATE: {
            SgdArgs a{};
            a.w = const_cast<float*>(wf(0));                      // caller-owned, updated in place
            a.g = buf(nd.preds[0]), a.flag = buf(v);
            a.lr = nd.p.lr, a.offset = nd.p.slice_lo[0], a.total = nd.p.cout;
            set_kernel<KID_SGD>(t, a, ceil_div(a.total, kBlock));
            break;
        }
        default:
            return g->fail(NG_EINVAL, "node %d: operator %d has no kernel", v, nd.op);
    }
    if (t.ntiles <= 0 || t.ntiles >= (1L << 31)) return g->fail(NG_ESHAPE, "node %d: %ld tiles cannot be launched", v, t.ntiles);
    return NG_OK;
}

}  // namespace ng
