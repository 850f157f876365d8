// The tile functions of every kernel and the table that names them (included by the files that build kernels from them).
//
// GPU tasks of the AoT multi-stream DAG executor: fp32 NCHW kernels for gfx950 (wave64).
//
// The Nimble paper (arXiv 2012.02732) ships no kernels of its own: it replays the base
// framework's operators unchanged (Section 5, "Experimental Setup"). These are the
// operators of its benchmark networks, written for CDNA4.
//
// Every operator is written once as a *tile function*: the share of 256 threads,
// addressed by a linear tile index. Two kinds of kernels are built from them:
//   * one stand-alone kernel per tile function (grid = number of tiles, 256 threads),
//     taking ONE by-value argument struct so that the task table can hold a ready-made
//     argument block per task (Section 4.1: kernel arguments are prepared once, ahead of time);
//   * the device-resident replay kernel (ng_resident.hip), in which persistent
//     workgroups of 512 threads (two tiles at a time) walk the recorded task schedule
//     themselves.
//
// Sizing rule that differs from usual throughput tuning: tasks are small (tens of
// thousands of elements) and are meant to run next to sibling tasks of other streams
// (Section 2, "GPU Streams"), so grids are sized by the work, never "fill the chip".
#pragma once
#include <hip/hip_runtime.h>
#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>
#include "ng_device.h"
#include "ng_internal.h"

namespace ng {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Access helpers. `far` is a compile-time constant at every call site. A far access is a
// device-scope access (sc1): it is served by the memory side, past the XCD-private L2, which
// is what makes a tensor written on one XCD readable on another without flushing or
// invalidating either L2. Far accesses go through buffer instructions (uniform tensor base
// + 32-bit byte offset), which carry the cache policy and come in 128-bit form; tensors are
// far smaller than the 4 GiB a 32-bit offset spans.
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
constexpr int kPolicyDeviceScope = 16;                       // cache-policy operand: sc1

__device__ __forceinline__ __amdgpu_buffer_rsrc_t tensor_rsrc(const float* base) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, 0x7FFFFFFF, 0x00020000);
}
__device__ __forceinline__ unsigned byte_offset(const float* base, const float* p) {
    return (unsigned)(reinterpret_cast<const char*>(p) - reinterpret_cast<const char*>(base));
}
// base: wave-uniform start of the tensor; p: this lane's address inside it
__device__ __forceinline__ float ldg(const float* base, const float* p, bool far) {
    if (!far) return *p;
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(tensor_rsrc(base), byte_offset(base, p), 0, kPolicyDeviceScope));
}
__device__ __forceinline__ float4 ldg4(const float* base, const float* p, bool far) {
    if (!far) return *reinterpret_cast<const float4*>(p);
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(tensor_rsrc(base), byte_offset(base, p), 0, kPolicyDeviceScope);
    float4 f;
    __builtin_memcpy(&f, &v, sizeof f);                     // the whole vector at once: extracting elements one by
    return f;                                               // one makes this compiler shrink the load to one dword
}
__device__ __forceinline__ void stg(float* base, float* p, float v, bool far) {
    if (!far) {
        *p = v;
        return;
    }
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), tensor_rsrc(base), byte_offset(base, p), 0, kPolicyDeviceScope);
}
__device__ __forceinline__ void stg4(float* base, float* p, float4 v, bool far) {
    if (!far) {
        *reinterpret_cast<float4*>(p) = v;
        return;
    }
    u32x4 u;
    __builtin_memcpy(&u, &v, sizeof u);
    __builtin_amdgcn_raw_buffer_store_b128(u, tensor_rsrc(base), byte_offset(base, p), 0, kPolicyDeviceScope);
}
// 128 bits at an address that is only a multiple of four bytes (rows or planes that are no multiple of four floats)
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ float4 ldg4_any(const float* base, const float* p, bool far) {
    if (far) return ldg4(base, p, true);
    const f32x4_any v = *reinterpret_cast<const f32x4_any*>(p);
    return make_float4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ void stg4_any(float* base, float* p, float4 v, bool far) {
    if (far) stg4(base, p, v, true);
    else *reinterpret_cast<f32x4_any*>(p) = f32x4_any{v.x, v.y, v.z, v.w};
}
// per-lane tensor (concat picks its source per lane): single relaxed device-scope accesses
__device__ __forceinline__ float ldg_any(const float* p, bool far) {
    return far ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p;
}
// 128-bit device-scope load from a per-lane address (16-byte aligned). The compiler does not
// know about loads issued from inline assembly, so the wait for the data is part of it.
__device__ __forceinline__ float4 ldg4_any_far(const float* p) {
    f32x4 v;
    asm volatile("global_load_dwordx4 %0, %1, off sc1\n\ts_waitcnt vmcnt(0)" : "=v"(v) : "v"(p) : "memory");
    return make_float4(v[0], v[1], v[2], v[3]);
}

// LDS floats every workgroup owns: the largest user is the conv3x3 input patch of the vector-ALU kernel (4 x 33 x 34).
constexpr int kSmemFloats = 5120;
// ... and what the patch-stationary kernels get instead: 24 floats (16 channels in three bf16 parts) for every pixel of their patches,
// 640 at most. Stand-alone kernels: only they; the resident kernel: every workgroup of the build that contains them.
constexpr int kSmemFloatsPatch = 24 * 256, kSmemFloatsWide = 24 * 640;
constexpr int smem_floats(int kid) {
    return is_c3_patch(kid) ? 24 * c3_patches(kid) * c3_patch_pixels(kid) : kid == KID_PW_P32 ? 2 * kSmemFloatsPatch : is_pw_patch(kid) ? kSmemFloatsPatch : kSmemFloats;
}

// ------------------------------------------------------------------------------------
// bn_act / relu: y = x * s[c] + t[c] (s, t folded from gamma, beta, mean, var), optional ReLU
// ------------------------------------------------------------------------------------
__device__ __forceinline__ void bn_coeff(const BnArgs& a, int c, float& s, float& t) {
    if (a.scale) {
        s = a.scale[c];
        t = a.shift[c];
    } else {
        s = 1.f;
        t = 0.f;
    }
}

// Every tile function takes a `wait` object and calls it exactly once, on every path and by
// every thread of the workgroup (it may contain a workgroup barrier), before the first access
// to data another task produced. Whatever does not depend on such data - index arithmetic,
// reading weights and coefficients - goes before the call, so that it overlaps with waiting
// for the producers. Stand-alone kernels pass NoWait; the resident kernel passes the wait
// for the task's completion counters, which does its work on the first call only.
// A convolution tile with a fused add_n calls `late` the same way, once, before it reads the
// other operands of the sum.
// A tile function meets the same number of workgroup barriers whatever its tile index and whether
// or not it is `live`: in the resident kernel two sub-blocks of one workgroup run different tiles
// of a task side by side and share every barrier.
struct NoWait {
    __device__ __forceinline__ void operator()() const {}
    __device__ __forceinline__ void late() const {}
    __device__ __forceinline__ constexpr bool far_out() const { return false; }
};

// Store one convolution result and, if a batch-norm / ReLU task was fused into the tile, that
// task's result as well (the kernels for larger problems: coefficients are fetched here, per
// value; the 16-row kernels fetch theirs before they wait for their inputs).
__device__ __forceinline__ void store_with_epilogue(float* y, const Epilogue& ep, size_t at, int channel, float v, bool fout) {
    stg(y, y + at, v, fout);
    if (ep.y != nullptr) {
        float s = 1.f, t = 0.f;
        if (ep.scale != nullptr) s = ep.scale[channel], t = ep.shift[channel];
        const float z = fmaf(v, s, t);
        stg(ep.y, ep.y + at, ep.relu ? fmaxf(z, 0.f) : z, fout);
    }
}

// The add_n epilogue of a convolution tile: v holds this lane's values (4 consecutive pixels if
// VEC, else one), `at` their position in the tensors; the sum runs in argument order.
template <bool VEC>
__device__ __forceinline__ void add_epilogue(const AddEpilogue& ea, float4 v, size_t at, bool fout) {
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int j = 0; j < kEpilogueAddMax; ++j) {               // constant indices only: the argument block stays in scalar registers
        if (j >= ea.k) break;
        float4 t = v;
        if (j != ea.zpos) {
            const float* x = j > ea.zpos ? ea.x[j > 0 ? j - 1 : 0] : ea.x[j < kEpilogueAddMax - 1 ? j : kEpilogueAddMax - 2];
            if (VEC) t = ldg4(x, x + at, ea.far != 0);
            else t.x = ldg(x, x + at, ea.far != 0);
        }
        if (j == 0) acc = t;
        else acc.x += t.x, acc.y += t.y, acc.z += t.z, acc.w += t.w;
    }
    if (VEC) stg4(ea.y, ea.y + at, acc, fout);
    else stg(ea.y, ea.y + at, acc.x, fout);
}

// Elementwise operators come in four partitions of the output into tiles, so that an
// elementwise task can take over the partition of the task that feeds it (then tile i of
// the consumer reads only what tile i of the producer wrote, and a workgroup that ran the
// one can run the other without waiting for anybody else):
//   PART_L256  tile t = elements [256 t, 256 t + 256), one per thread (pool, dwconv order)
//   PART_L1024 tile t = elements [1024 t, 1024 t + 1024), one float4 per thread
//   PART_R64   tile t = 16 channels x 64 columns (column = image * HW + pixel), the tile of
//              the 128-bit conv1x1; thread = (channel tid / 16, 4 columns from 4 (tid % 16))
//   PART_R16   tile t = 16 channels x 16 columns, the tile of the 32-bit conv1x1
// ElemIndex: first element a thread owns (VEC of them, consecutive), its channel, validity.
struct ElemIndex {
    int e, c;
    bool ok;
};
template <int PART>
__device__ __forceinline__ ElemIndex elem_index(int tile, int tid, int C, int HW, int total, int cols) {
    ElemIndex r;
    if (PART == PART_L1024 || PART == PART_L256) {
        r.e = (tile * kBlock + tid) * (PART == PART_L1024 ? 4 : 1);
        r.ok = r.e < total;
        r.c = (r.e / HW) % C;
    } else {
        constexpr int TN = PART == PART_R64 ? 64 : 16, V = PART == PART_R64 ? 4 : 1;
        const int tiles_n = (cols + TN - 1) / TN;
        const int by = tile / tiles_n, bx = tile - by * tiles_n;
        const int col = bx * TN + V * (tid & 15);
        r.c = by * 16 + (tid >> 4);
        r.ok = r.c < C && col < cols;
        const int img = col / HW, pix = col - img * HW;
        r.e = (img * C + r.c) * HW + pix;
    }
    return r;
}

template <int PART, bool FIN, class Wait>
__device__ __forceinline__ void bn_act_tile(const BnArgs& a, int tile, float*, int tid, bool live, Wait& wait) {
    const bool fout = wait.far_out();       // device-scope stores: some reader of the result sits on another XCD
    const ElemIndex ix = elem_index<PART>(tile, tid, a.C, a.HW, a.total, a.cols);
    const bool active = live && ix.ok;
    float s = 1.f, t = 0.f;
    if (active) bn_coeff(a, ix.c, s, t);
    wait();
    if (!active) return;
    if (PART == PART_L1024 || PART == PART_R64) {          // HW % 4 == 0: a float4 never straddles channels
        float4 v = ldg4(a.x, a.x + ix.e, FIN);
        v.x = fmaf(v.x, s, t), v.y = fmaf(v.y, s, t), v.z = fmaf(v.z, s, t), v.w = fmaf(v.w, s, t);
        if (a.relu) v.x = fmaxf(v.x, 0.f), v.y = fmaxf(v.y, 0.f), v.z = fmaxf(v.z, 0.f), v.w = fmaxf(v.w, 0.f);
        stg4(a.y, a.y + ix.e, v, fout);
    } else {
        const float v = fmaf(ldg(a.x, a.x + ix.e, FIN), s, t);
        stg(a.y, a.y + ix.e, a.relu ? fmaxf(v, 0.f) : v, fout);
    }
}

// ------------------------------------------------------------------------------------
// add_n: elementwise sum of k tensors, accumulated in argument order
// ------------------------------------------------------------------------------------
template <int PART, bool FIN, class Wait>
__device__ __forceinline__ void add_n_tile(const AddArgs& a, int tile, float*, int tid, bool live, Wait& wait) {
    const bool fout = wait.far_out();       // device-scope stores: some reader of the result sits on another XCD
    const ElemIndex ix = elem_index<PART>(tile, tid, a.C, a.HW, a.total, a.cols);
    wait();
    if (!live || !ix.ok) return;
    const int e = ix.e;
    if (PART == PART_L1024 || PART == PART_R64) {
        float4 acc = ldg4(a.x[0], a.x[0] + e, FIN);
#pragma unroll
        for (int j = 1; j < NG_MAX_PREDS; ++j) {
            if (j >= a.k) break;
            const float4 v = ldg4(a.x[j], a.x[j] + e, FIN);
            acc.x += v.x, acc.y += v.y, acc.z += v.z, acc.w += v.w;
        }
        stg4(a.y, a.y + e, acc, fout);
    } else {
        float acc = ldg(a.x[0], a.x[0] + e, FIN);
#pragma unroll
        for (int j = 1; j < NG_MAX_PREDS; ++j) {
            if (j >= a.k) break;
            acc += ldg(a.x[j], a.x[j] + e, FIN);
        }
        stg(a.y, a.y + e, acc, fout);
    }
}

// ------------------------------------------------------------------------------------
// concat: output channel block j = channels [lo_j, lo_j + cnt_j) of input j
// ------------------------------------------------------------------------------------
template <bool VEC4, bool FIN, class Wait>
__device__ __forceinline__ void concat_tile(const ConcatArgs& a, int tile, float*, int tid, bool live, Wait& wait) {
    const bool fout = wait.far_out();       // device-scope stores: some reader of the result sits on another XCD
    const int i = tile * kBlock + tid;
    const int e = VEC4 ? i * 4 : i;
    const bool active = live && e < a.total;
    const int plane = e / a.HW, pix = e - plane * a.HW;
    const int n = plane / a.C, c = plane - n * a.C;
    const float* base = a.x[0];
    int cin = a.cin[0], lo = a.lo[0], first = a.first[0];
#pragma unroll
    for (int q = 1; q < NG_MAX_PREDS; ++q)
        if (q < a.k && c >= a.first[q]) base = a.x[q], cin = a.cin[q], lo = a.lo[q], first = a.first[q];
    const float* src = base + ((size_t)(n * cin + lo + c - first)) * a.HW + pix;
    wait();
    if (!active || src == a.y + e) return;                   // an input the memory plan placed inside the result is there already
    if (VEC4) {
        float4 v;
        if (FIN) v = ldg4_any_far(src);
        else v = *reinterpret_cast<const float4*>(src);
        stg4(a.y, a.y + e, v, fout);
    } else {
        stg(a.y, a.y + e, ldg_any(src, FIN), fout);
    }
}

// ------------------------------------------------------------------------------------
// pool3x3: max (out-of-bounds taps ignored) or average over the in-bounds taps
// ------------------------------------------------------------------------------------
// Windowed kernels: a tile is 256 P consecutive outputs, thread t owns outputs t, t + 256, ...
// of it (P = 1 for stand-alone launches; P = 4 when a task would otherwise need several
// rounds on the workgroups of its stream - one round costs one trip to memory however many
// loads are in flight, and 1024 consecutive outputs are also the tile of the float4
// elementwise kernels, which can then take over the partition).
template <int P, bool EA, bool FIN, class Wait>
__device__ __forceinline__ void pool3x3_tile(const typename std::conditional<EA, PoolAddArgs, PoolArgs>::type& a, int tile, float*, int tid,
                                             bool live, Wait& wait) {
    const bool fout = wait.far_out();       // device-scope stores: some reader of the result sits on another XCD
    const int base = tile * kBlock * P + tid;
    const bool active = live && base < a.total;
    // all taps of all P outputs are loaded unconditionally from clamped coordinates, so the
    // loads are independent and in flight together; taps outside the image are masked afterwards
    float v[P][9];
    int r0[P], c0[P];
    const float* src[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int i = min(base + p * kBlock, a.total - 1);
        const int ow = i % a.Wo, t = i / a.Wo;
        const int oh = t % a.Ho, plane = t / a.Ho;
        src[p] = a.x + (size_t)plane * a.H * a.W;
        r0[p] = oh * a.stride - a.pad, c0[p] = ow * a.stride - a.pad;
    }
    wait();
    if (!EA && !active) return;                              // with a fused add_n every thread goes on to the late wait
    float res[P];
    if (active) {
#pragma unroll
        for (int p = 0; p < P; ++p) {
#pragma unroll
            for (int dr = 0; dr < 3; ++dr)
#pragma unroll
                for (int dc = 0; dc < 3; ++dc)
                    v[p][dr * 3 + dc] = ldg(a.x, src[p] + min(max(r0[p] + dr, 0), a.H - 1) * a.W + min(max(c0[p] + dc, 0), a.W - 1), FIN);
        }
        __builtin_amdgcn_sched_barrier(0);                   // all loads are issued before the first use
#pragma unroll
        for (int p = 0; p < P; ++p) {
            float acc = a.mode == 0 ? -INFINITY : 0.f;
            int cnt = 0;
#pragma unroll
            for (int dr = 0; dr < 3; ++dr)
#pragma unroll
                for (int dc = 0; dc < 3; ++dc) {
                    const int r = r0[p] + dr, c = c0[p] + dc;
                    const bool in = r >= 0 && r < a.H && c >= 0 && c < a.W;
                    if (a.mode == 0) acc = in ? fmaxf(acc, v[p][dr * 3 + dc]) : acc;
                    else acc += in ? v[p][dr * 3 + dc] : 0.f;
                    cnt += in;
                }
            res[p] = a.mode == 0 ? acc : acc / (float)cnt;
            if (base + p * kBlock < a.total) stg(a.y, a.y + base + p * kBlock, res[p], fout);
        }
    }
    if constexpr (EA) {
        wait.late();
        if (active) {
#pragma unroll
            for (int p = 0; p < P; ++p)
                if (base + p * kBlock < a.total)
                    add_epilogue<false>(a.ea, make_float4(res[p], 0.f, 0.f, 0.f), (size_t)(base + p * kBlock), fout);
        }
    }
}

// ------------------------------------------------------------------------------------
// dwconv: depthwise K x K, pad K/2, stride S; P outputs per thread
// ------------------------------------------------------------------------------------
template <int K, int S, int P, bool FIN, class Wait>
__device__ __forceinline__ void dwconv_tile(const DwArgs& a, int tile, float*, int tid, bool live, Wait& wait) {
    const bool fout = wait.far_out();       // device-scope stores: some reader of the result sits on another XCD
    const int base = tile * kBlock * P + tid;
    const bool active = live && base < a.total;
    // unconditional loads from clamped coordinates (all in flight together), masked afterwards
    float v[P][K * K], w[P][K * K];
    int r0[P], c0[P];
    const float* src[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int i = min(base + p * kBlock, a.total - 1);
        const int ow = i % a.Wo, t = i / a.Wo;
        const int oh = t % a.Ho, plane = t / a.Ho;
        src[p] = a.x + (size_t)plane * a.H * a.W;
        const float* wt = a.w + (plane % a.C) * K * K;
        r0[p] = oh * S - K / 2, c0[p] = ow * S - K / 2;
#pragma unroll
        for (int q = 0; q < K * K; ++q) w[p][q] = wt[q];       // filter taps: not produced by any task
    }
    wait();
    if (!active) return;
#pragma unroll
    for (int p = 0; p < P; ++p) {
#pragma unroll
        for (int dr = 0; dr < K; ++dr)
#pragma unroll
            for (int dc = 0; dc < K; ++dc)
                v[p][dr * K + dc] = ldg(a.x, src[p] + min(max(r0[p] + dr, 0), a.H - 1) * a.W + min(max(c0[p] + dc, 0), a.W - 1), FIN);
    }
    __builtin_amdgcn_sched_barrier(0);                       // all loads are issued before the first use
#pragma unroll
    for (int p = 0; p < P; ++p) {
        float acc = 0.f;
#pragma unroll
        for (int dr = 0; dr < K; ++dr)
#pragma unroll
            for (int dc = 0; dc < K; ++dc) {
                const int r = r0[p] + dr, cc = c0[p] + dc;
                const bool in = r >= 0 && r < a.H && cc >= 0 && cc < a.W;
                acc = fmaf(w[p][dr * K + dc], in ? v[p][dr * K + dc] : 0.f, acc);
            }
        if (base + p * kBlock < a.total) stg(a.y, a.y + base + p * kBlock, acc, fout);
    }
}

// ------------------------------------------------------------------------------------
// global_avgpool: one wavefront per (n, c) plane, reduction across 64 lanes
// ------------------------------------------------------------------------------------
// Sum over the 64 lanes of a wavefront with data-parallel-primitive moves (one vector instruction per step, no trip
// through the LDS crossbar as a shuffle takes): a scan inside each row of 16 lanes (shifts by 1, 2, 4, 8, zeros shifted
// in) leaves a row's sum in its lane 15; lane 15 of rows 0 and 2 is then added to rows 1 and 3, lane 31 to rows 2 and 3,
// and lane 63 holds the total, which every lane gets back. The order of the additions is fixed.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_add(float v) {
    const int moved = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROW_MASK, 0xf, true);
    return v + __builtin_bit_cast(float, moved);
}
__device__ __forceinline__ float wave_sum(float v) {
    v = dpp_add<0x111, 0xf>(v);                              // row_shr:1
    v = dpp_add<0x112, 0xf>(v);                              // row_shr:2
    v = dpp_add<0x114, 0xf>(v);                              // row_shr:4
    v = dpp_add<0x118, 0xf>(v);                              // row_shr:8
    v = dpp_add<0x142, 0xa>(v);                              // row_bcast:15 into rows 1 and 3
    v = dpp_add<0x143, 0xc>(v);                              // row_bcast:31 into rows 2 and 3
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

template <bool FIN, class Wait>
__device__ __forceinline__ void global_avgpool_tile(const GapArgs& a, int tile, float*, int tid, bool live, Wait& wait) {
    const bool fout = wait.far_out();       // device-scope stores: some reader of the result sits on another XCD
    wait();
    const int lane = tid & 63;
    const int plane = tile * (kBlock / 64) + (tid >> 6);
    if (!live || plane >= a.planes) return;
    const float* src = a.x + (size_t)plane * a.HW;
    float acc = 0.f;
    for (int p = lane; p < a.HW; p += 64) acc += ldg(a.x, src + p, FIN);
    acc = wave_sum(acc);
    if (lane == 0) stg(a.y, a.y + plane, acc / (float)a.HW, fout);
}

// ------------------------------------------------------------------------------------
// fc (small batch): one wavefront per output feature; y[n][o] = <W[o], x[n]> + b[o]
// ------------------------------------------------------------------------------------
template <bool FIN, class Wait>
__device__ __forceinline__ void fc_gemv_tile(const FcArgs& a, int tile, float*, int tid, bool live, Wait& wait) {
    const bool fout = wait.far_out();       // device-scope stores: some reader of the result sits on another XCD
    wait();
    const int lane = tid & 63;
    const int o = tile * (kBlock / 64) + (tid >> 6);
    if (!live || o >= a.Cout) return;
    const float* wr = a.w + (size_t)o * a.Cin;
    for (int n = 0; n < a.N; ++n) {
        const float* xr = a.x + (size_t)n * a.Cin;
        float acc = 0.f;
        if ((a.Cin & 3) == 0) {
            for (int k = lane * 4; k < a.Cin; k += 256) {
                const float4 wv = *reinterpret_cast<const float4*>(wr + k);
                const float4 xv = ldg4(a.x, xr + k, FIN);
                acc = fmaf(wv.x, xv.x, acc), acc = fmaf(wv.y, xv.y, acc);
                acc = fmaf(wv.z, xv.z, acc), acc = fmaf(wv.w, xv.w, acc);
            }
        } else {
            for (int k = lane; k < a.Cin; k += 64) acc = fmaf(wr[k], ldg(a.x, xr + k, FIN), acc);
        }
        acc = wave_sum(acc);
        if (lane == 0) stg(a.y, a.y + (size_t)n * a.Cout + o, acc + a.b[o], fout);
    }
}

// ------------------------------------------------------------------------------------
// conv1x1 (and large-batch fc) on the matrix cores: Y[Cout x cols] = W[Cout x Cin] * X[Cin x cols]
// with cols = N * HW. v_mfma_f32_16x16x4_f32: A fragment lane l -> A[l % 16][l / 16],
// B fragment lane l -> B[l / 16][l % 16], accumulator register r of lane l -> D[4 * (l / 16) + r][l % 16].
// A workgroup of four wavefronts (2 x 2) owns a TM x TN output tile; K is walked in
// slices of KC staged through LDS, A as [k][m] so both fragments read rows. The weights are
// repacked at bind time into that order, W^T[CinP][CoutP] (zero padded; CinP a multiple of
// KC, CoutP of TM), so a slice of them is read and stored along m without any mask. Rows of
// the LDS slices are 16 (mod 32) floats apart: the four 16-lane groups of a wavefront, which
// read four consecutive rows, then hit different banks.
// ------------------------------------------------------------------------------------
template <int TM, int TN, int KC, bool FIN, class Wait>
__device__ __forceinline__ void conv1x1_mfma_tile(const PwArgs& a, int tile, float* smem, int tid, bool live, Wait& wait) {
    const bool fout = wait.far_out();       // device-scope stores: some reader of the result sits on another XCD
    wait();
    constexpr int WM = TM / 2, WN = TN / 2;           // per-wavefront sub-tile
    constexpr int FM = WM / 16, FN = WN / 16;         // 16 x 16 fragments per wavefront
    constexpr int LDA = TM + 16, LDB = TN + 16;
    static_assert(LDA % 32 == 16 && LDB % 32 == 16, "row pitch of the LDS slices");
    static_assert(KC * (LDA + LDB) <= kSmemFloats, "LDS budget");
    static_assert(kBlock % TM == 0 && kBlock % TN == 0 && KC % (kBlock / TM) == 0 && KC % (kBlock / TN) == 0, "fill pattern");
    float* As = smem;                                 // [KC][LDA]
    float* Bs = smem + KC * LDA;                      // [KC][LDB]

    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int by = tile / a.tiles_n, bx = tile - by * a.tiles_n;
    const int m0 = by * TM, n0 = bx * TN;

    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // A slice: W^T[k0 + k][m0 + m] -> As[k][m]; B slice: X[k0 + k][n0 + n] -> Bs[k][n]; consecutive
    // threads walk m and the pixels. Loads of X are unconditional from clamped indices (independent,
    // all in flight), zeroed when they are stored. The loads of slice k0 + KC are issued before the
    // matrix instructions of slice k0 and stored after them, so their latency overlaps with the arithmetic.
    constexpr int RA = kBlock / TM;                           // k rows of A covered per pass
    constexpr int RK = kBlock / TN;                           // k rows of B covered per pass
    const int CoutP = (a.Cout + TM - 1) / TM * TM;
    const float* wcol = a.wp + m0 + tid % TM + (size_t)(tid / TM) * CoutP;
    const int fn = tid % TN, fcol = n0 + fn;
    const int fccol = min(fcol, a.cols - 1);
    const int fimg = fccol / a.HW, fpix = fccol - fimg * a.HW;
    const float* xc = a.x + (size_t)fimg * a.Cin * a.HW + fpix;
    float va[KC / RA], vb[KC / RK];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int p = 0; p < KC / RA; ++p) va[p] = wcol[(size_t)(k0 + p * RA) * CoutP];
#pragma unroll
        for (int p = 0; p < KC / RK; ++p) vb[p] = ldg(a.x, xc + (size_t)min(k0 + tid / TN + p * RK, a.Cin - 1) * a.HW, FIN);
    };
    if (live) fetch(0);
    for (int k0 = 0; k0 < a.Cin; k0 += KC) {
        if (live) {
#pragma unroll
            for (int p = 0; p < KC / RA; ++p) As[(tid / TM + p * RA) * LDA + tid % TM] = va[p];
#pragma unroll
            for (int p = 0; p < KC / RK; ++p) {
                const int k = tid / TN + p * RK;
                Bs[k * LDB + fn] = (fcol < a.cols && k0 + k < a.Cin) ? vb[p] : 0.f;
            }
        }
        __syncthreads();
        if (live && k0 + KC < a.Cin) fetch(k0 + KC);
        if (live)
#pragma unroll
        for (int kk = 0; kk < KC; kk += 4) {
            float af[FM], bf[FN];
#pragma unroll
            for (int i = 0; i < FM; ++i) af[i] = As[(kk + (lane >> 4)) * LDA + wm * WM + i * 16 + (lane & 15)];
#pragma unroll
            for (int j = 0; j < FN; ++j) bf[j] = Bs[(kk + (lane >> 4)) * LDB + wn * WN + j * 16 + (lane & 15)];
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[i], bf[j], acc[i][j], 0, 0, 0);
        }
        __syncthreads();
    }

#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int col = n0 + wn * WN + j * 16 + (lane & 15);
            if (col >= a.cols || !live) continue;
            const int img = col / a.HW, pix = col - img * a.HW;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = m0 + wm * WM + i * 16 + 4 * (lane >> 4) + r;
                if (m < a.Cout) {
                    const float b = a.bias ? a.bias[m] : 0.f;
                    store_with_epilogue(a.y, a.ep, ((size_t)img * a.Cout + m) * a.HW + pix, m, acc[i][j][r] + b, fout);
                }
            }
        }
}

// ------------------------------------------------------------------------------------
// conv3x3 with many output columns (large maps, batches): the LDS-staged scheme of the kernel
// above on the implicit GEMM Y[Cout x cols] = W'[Cout x K'] * P[K' x cols], with K ordered tap
// first: k' = tap * CinP + ci, CinP = Cin rounded up to a multiple of KC. A K slice then has
// ONE tap, so where the slice's patch rows lie relative to a column (and whether that is inside
// the image) is worked out once per slice and thread, and the rows differ by a channel stride.
// The weights are repacked at bind time into W'^T[k'][CoutP] (zero padded; CoutP a multiple of
// TM), so a slice of them is read and stored to LDS along m without any mask. Rows of the LDS
// slices are 16 (mod 32) floats apart: the four 16-lane groups of a wavefront, which read four
// consecutive rows, then hit different banks. Every patch element is read from global memory
// once per workgroup tile instead of once per 16 x 16 MFMA tile.
// ------------------------------------------------------------------------------------
template <int TM, int TN, int KC, bool FIN, class Wait>
__device__ __forceinline__ void conv3x3_lds_tile(const C3Args& a, int tile, float* smem, int tid, bool live, Wait& wait) {
    const bool fout = wait.far_out();       // device-scope stores: some reader of the result sits on another XCD
    constexpr int WM = TM / 2, WN = TN / 2;           // per-wavefront sub-tile
    constexpr int FM = WM / 16, FN = WN / 16;         // 16 x 16 fragments per wavefront
    constexpr int LDA = TM + 16, LDB = TN + 16;
    static_assert(LDA % 32 == 16 && LDB % 32 == 16, "row pitch of the LDS slices");
    static_assert(KC * (LDA + LDB) <= kSmemFloats, "LDS budget");
    static_assert(kBlock % TM == 0 && kBlock % TN == 0 && KC % (kBlock / TM) == 0 && KC % (kBlock / TN) == 0, "fill pattern");
    float* As = smem;                                 // [KC][LDA]
    float* Bs = smem + KC * LDA;                      // [KC][LDB]

    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int by = tile / a.tiles_n, bx = tile - by * a.tiles_n;
    const int m0 = by * TM, n0 = bx * TN;
    const int CinP = a.groups, CoutP = (a.Cout + TM - 1) / TM * TM;
    const int HWo = a.Ho * a.Wo, HW = a.H * a.W;
    // the column this thread fills in every B slice
    const int fill_col = n0 + tid % TN;
    const int ccol = min(fill_col, a.cols - 1);
    const int fimg = ccol / HWo, fpix = ccol - fimg * HWo;
    const int foy = fpix / a.Wo, fox = fpix - foy * a.Wo;
    const int iy0 = foy * a.stride - a.pad, ix0 = fox * a.stride - a.pad;
    const float* xin = a.x + (size_t)fimg * a.Cin * HW;
    // the weight column this thread fills in every A slice
    constexpr int RA = kBlock / TM, RB = kBlock / TN;            // k rows covered per pass
    const float* wcol = a.wp + m0 + tid % TM + (size_t)(tid / TM) * CoutP;

    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    wait();

    for (int tap = 0; tap < 9; ++tap) {
        const int dr = tap / 3, dc = tap - 3 * dr;
        const int iy = iy0 + dr, ix = ix0 + dc;
        const bool inside = fill_col < a.cols && (unsigned)iy < (unsigned)a.H && (unsigned)ix < (unsigned)a.W;
        const float* xtap = xin + min(max(iy, 0), a.H - 1) * a.W + min(max(ix, 0), a.W - 1);
        for (int c0 = 0; c0 < CinP; c0 += KC) {
            if (live) {
                float v[KC / RA], pv[KC / RB];
                const float* wk = wcol + (size_t)(tap * CinP + c0) * CoutP;
#pragma unroll
                for (int p = 0; p < KC / RA; ++p) v[p] = wk[(size_t)p * RA * CoutP];
#pragma unroll
                for (int p = 0; p < KC / RB; ++p) pv[p] = ldg(a.x, xtap + (size_t)min(c0 + tid / TN + p * RB, a.Cin - 1) * HW, FIN);
                __builtin_amdgcn_sched_barrier(0);               // all loads of the slice are issued before the first use
#pragma unroll
                for (int p = 0; p < KC / RA; ++p) As[(tid / TM + p * RA) * LDA + tid % TM] = v[p];
#pragma unroll
                for (int p = 0; p < KC / RB; ++p) {
                    const int kk = tid / TN + p * RB;
                    Bs[kk * LDB + tid % TN] = (inside && c0 + kk < a.Cin) ? pv[p] : 0.f;
                }
            }
            __syncthreads();
            if (live)
#pragma unroll
            for (int kk = 0; kk < KC; kk += 4) {
                float af[FM], bf[FN];
#pragma unroll
                for (int i = 0; i < FM; ++i) af[i] = As[(kk + (lane >> 4)) * LDA + wm * WM + i * 16 + (lane & 15)];
#pragma unroll
                for (int j = 0; j < FN; ++j) bf[j] = Bs[(kk + (lane >> 4)) * LDB + wn * WN + j * 16 + (lane & 15)];
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[i], bf[j], acc[i][j], 0, 0, 0);
            }
            __syncthreads();
        }
    }

#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int col = n0 + wn * WN + j * 16 + (lane & 15);
            if (col >= a.cols || !live) continue;
            const int img = col / HWo, pix = col - img * HWo;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = m0 + wm * WM + i * 16 + 4 * (lane >> 4) + r;
                if (m < a.Cout) store_with_epilogue(a.y, a.ep, ((size_t)img * a.Cout + m) * HWo + pix, m, acc[i][j][r], fout);
            }
        }
}

// ------------------------------------------------------------------------------------
// fp32 products on the bf16 matrix cores. A value is split into three bf16 parts, x = h + m + l: h the upper half of its bits, m
// the rest rounded to nearest even, l what is left of it (24 = 8 + 8 + 8 bits: exact). Of the nine products of two split values
// the six of 2^-16 and larger are formed: h h in an accumulator of its own, h m, m h, m m, h l and l h in a second one, added
// once at the end. v_mfma_f32_32x32x16_bf16 does 16 times the work of v_mfma_f32_16x16x4_f32 per cycle, six of them
// replace sixteen cycles by six. The large accumulator is rounded once per 16 k instead of once per 4 k, so that the results
// are closer to 64 bits than those of the fp32 instructions: 2-norm of the error over that of the result, K = 288 - 4032:
// 0.7 - 2.7e-7 against 2.2 - 7.6e-7. (All six in one accumulator: 2.3 - 8.3e-7, which is why there are two.)
// Small values: bf16 has the exponents of fp32 and a quantum of 2^-133, and m and l lie 2^-8 and 2^-16 below x. All 24 bits are
// there down to |x| = 2^-110, on either side of the product; below that x is taken to the next multiple of 2^-133 (2-norm of
// the error for values around 2^-118: 9e-6, 2^-126: 2e-3; the fp32 instructions lose nothing there). Sums that also have
// values of 2^-110 and more do not notice. Parts scaled by 64 and 4096 would keep all bits down to 2^-122, but take an
// accumulator more and two multiplications per activation: conv3x3 1 - 3 % and conv1x1 up to 8 % slower, an Inception-style network
// at batch 1, 6 and 32 711 -> 725, 1151 -> 1170, 3613 -> 3633 us; and the full build of the resident kernel spills 622 registers
// instead of 184 (a network of sixteen conv3x3_mfma_split_k, 28 x 28 128 and below, 386 -> 552 us; with two slices of weights
// ahead there instead of three 208 registers and 447 us).
// The method: G. Henry, P. T. P. Tang, A. Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For
// Higher-Precision Computations", 2019.
// Infinities and NaN. h is finite wherever x is (its bits are cut off, not rounded up), infinite where x is, NaN where x is (a
// signalling NaN whose upper half is that of an infinity counts as one). So the sum of the h h has the infinities and NaNs that
// the fp32 products have; the lower parts of an infinity are NaN, so where the sum of the h h is not finite it is the result
// (split_sum). It is also where a sum outgrows fp32, which needs products whose magnitudes add up to more than the largest fp32 number.
// ------------------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// two values at a time: the parts of x0 in the low halves of h, m, l, those of x1 in the high halves
__device__ __forceinline__ void split_bf16x3(float x0, float x1, unsigned& h, unsigned& m, unsigned& l) {
    const unsigned b0 = __builtin_bit_cast(unsigned, x0), b1 = __builtin_bit_cast(unsigned, x1);
    h = __builtin_amdgcn_perm(b1, b0, 0x07060302);              // the upper halves of both
    const float r0 = x0 - __builtin_bit_cast(float, b0 & 0xffff0000u), r1 = x1 - __builtin_bit_cast(float, b1 & 0xffff0000u);
    m = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{r0, r1}), bf16x2));
    const float q0 = r0 - __builtin_bit_cast(float, m << 16), q1 = r1 - __builtin_bit_cast(float, m & 0xffff0000u);
    l = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{q0, q1}), bf16x2));
}
__device__ __forceinline__ void split8(const float (&v)[8], u32x4 (&part)[3]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        unsigned h, m, l;
        split_bf16x3(v[2 * q], v[2 * q + 1], h, m, l);
        part[0][q] = h, part[1][q] = m, part[2][q] = l;
    }
}
// 32 x 32 outputs, 16 k: high += ah bh, low += the five smaller products
__device__ __forceinline__ void mfma_split(const u32x4 (&a)[3], const u32x4 (&b)[3], f32x16& high, f32x16& low) {
    constexpr int pa[6] = {0, 2, 1, 0, 1, 0}, pb[6] = {0, 0, 1, 2, 0, 1};
#pragma unroll
    for (int p = 0; p < 6; ++p) {
        f32x16& d = p == 0 ? high : low;
        d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[pa[p]]), __builtin_bit_cast(bf16x8, b[pb[p]]), d, 0, 0, 0);
    }
}
__device__ __forceinline__ f32x16 split_sum(const f32x16& high, const f32x16& low) {
    f32x16 v;
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = __builtin_fabsf(high[q]) < __builtin_inff() ? high[q] + low[q] : high[q];
    return v;
}

// ------------------------------------------------------------------------------------
// conv3x3 for many output pixels (large maps, batches), patch-stationary: Y[Cout x pixels] = W[Cout x 9 Cin] * patches.
// A tile is TM output channels by a run of TN consecutive output pixels of one strip of an image: columns [x0, x0 + ws), row-major,
// so a run may wrap over several rows. Narrow images are one strip; wide ones are cut so that a run's patch fits into LDS
// (choose_strips; 64 pixels of a 147-wide image need 3 x 147 pixels of patch, of a 49-wide strip 197). K is walked in blocks
// of 16 input channels, and within a block tap by tap, in split bf16 (above):
//   * B operand. The input pixels the run needs - from its first pixel's upper left neighbour to its last one's lower right, rows of
//     the strip and its halo, the padding stored as zeros - are kept in LDS for one block of 16 channels, already split: three
//     planes, 32 bytes per pixel and plane. Lane (r, g) takes channels 8 g .. 8 g + 7 of pixel r with one 128-bit read per part;
//     which half of a pixel's 32 bytes holds which eight channels alternates every four pixels, so that eight lanes that are read
//     together hit all banks. A tap is an address shift (dr Wp + dc pixels): the nine taps of a block run off ONE patch without a
//     barrier between them, and each input element is fetched and split once per tile and block instead of once per tap.
//   * A operand. The weights were split and repacked at bind time into [block * 9 + tap][CoutP / 32][part][lane][8], so a
//     fragment is three 128-bit loads of 1 KiB in a row, straight from memory (L2) into registers, two or three slices ahead.
//   * Filling the patch: a thread owns up to 2 PM / 256 (pixel, 8 channels) items; their global offsets are worked out once
//     per tile (out-of-image and padding positions get an offset beyond the buffer's size, for which a buffer load returns
//     0), so a fill is eight 32-bit loads with a scalar channel offset and three 128-bit LDS writes per item. With two patches
//     (BUFFERS) the next block's is split and stored between the matrix instructions of this one: one barrier per block.
// A wavefront owns 32 rows x 64 pixels (PX = 2 blocks of 32), so a weight fragment (3 KiB through the vector L1) serves twelve matrix
// instructions. 64 rows x 128 pixels: 2 x 2 wavefronts. 64 x 64 and 32 x 128: two wavefronts side by side and K over two pairs (WK), by taps: of the nine
// of a block one pair takes five and the other four, in turns. 96 x 64: two wavefronts in each pair, of which one owns the upper 32 rows
// and the other the lower ones, and each one half of the middle rows.
// What bounds it is no one unit: by the counters of single launches of the layers of an Inception-style network at batch 32 matrix cores
// are busy in 32 - 37 % of the cycles (32 x 128: 24), LDS in 19 - 25 % (wide 64 x 64: 45), in more than half of those with conflicts, and
// memory moves up to 3.6 TB/s. Without the bank conflicts at the ends of
// rows, with half the barriers or three instead of two wavefronts per SIMD it takes the same time. Before, a wavefront owned 32 x 32
// (96 rows: 64 x 32), and wide images had patches of up to 640 pixels, whole rows. Layers at batch 32, us before and after: 147 x 147 32 -> 64
// 274 -> 256, 149 x 149 32 -> 32 165 -> 141, 73 x 73 80 -> 192 296 -> 282, 35 x 35 96 -> 96 59.8 -> 53.8, 35 x 35 288 -> 384 stride 2
// 150 -> 133, 17 x 17 192 -> 192 46.2 -> 44.1, 8 x 8 384 -> 768 73.5 -> 64.7; six images, 63 x 63 80 -> 192 59.8 -> 51.0. Two patches
// against one: 149 x 149 32 -> 32 147, 17 x 17 192 -> 192 44.3; for 64 x 128 and the wide 64 x 64 one is faster (256 against 280, 133 against 166:
// the strips that two patches have room for are too narrow).
// Needs Cin % 16 == 0 and a patch of at most PM pixels.
// ------------------------------------------------------------------------------------
template <int ROWS, int WN, int WK, int PX, int PM, int BUFFERS, bool FIN, class Wait>
__device__ __forceinline__ void conv3x3_patch_tile(const C3Args& a, int tile, float* smem, int tid, bool live, Wait& wait) {
    const bool fout = wait.far_out();
    constexpr int FM = ROWS == 96 ? 2 : 1, UNITS = FM + PX - 1, TM = ROWS, TN = 32 * PX * WN;
    constexpr int TAPS = WK == 1 ? 9 : 4, ST = WK == 1 ? 3 : 2;     // slices of every block that a wavefront has, and how far ahead it loads weights
    constexpr int ITEMS = (2 * PM + kBlock - 1) / kBlock, PLANE = 2 * PM;           // PLANE: one part of a patch, in units of 16 bytes
    constexpr int kIn = FIN ? kPolicyDeviceScope : 0;
    static_assert((ROWS == 96 ? 2 : ROWS / 32) * WN * WK == 4 && (PX == 2 || (WK == 1 && FM == 1)) && (WK == 1 || 4 * (8 + 8 * FM) * 64 <= BUFFERS * PM * 24), "four wavefronts; the sums that are handed over fit");
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 31, g = lane >> 5;
    const int by = tile % a.co_groups, bt = tile / a.co_groups;
    // the wavefront's share of K, and its blocks of the tile: rows `top` (96 rows: and the middle ones) x pixels n[0] and n[1]
    const int kg = WK == 2 ? wave >> 1 : 0, wm = ROWS == 64 ? (WK == 2 ? wave & 1 : wave >> 1) : ROWS == 96 ? wave & 1 : 0, wn = wave % WN;
    const int top = ROWS == 96 ? 2 * wm : wm;
    const int n[2] = {ROWS == 96 ? wm : PX * wn, ROWS == 96 ? 1 - wm : PX * wn + 1};
    const int img = bt / a.tiles_xy, seg = bt - img * a.tiles_xy;
    const int HWo = a.Ho * a.Wo, HW = a.H * a.W;
    // the strip of the image (all but the last are tiles_x wide) and the run of its pixels
    const int per_strip = (a.tiles_x * a.Ho + TN - 1) / TN, strip = seg / per_strip, x0 = strip * a.tiles_x, ws = min(a.tiles_x, a.Wo - x0);
    const int p0 = (seg - strip * per_strip) * TN, npx = min(TN, ws * a.Ho - p0);
    const int oy_a = p0 / ws, ox_a = p0 - oy_a * ws, oy_b = (p0 + npx - 1) / ws, ox_b = p0 + npx - 1 - oy_b * ws;
    // the patch: rows of Wp input pixels, from the first to the last one that the run needs, one after the other
    const int iy_a = oy_a * a.stride - a.pad, ix_a = x0 * a.stride - a.pad, Wp = (ws - 1) * a.stride + 3;
    const int skip = ox_a * a.stride, P = ((oy_b - oy_a) * a.stride + 2) * Wp + ox_b * a.stride + 3 - skip;
    const int blocks = a.groups / 16, Mf = a.co_groups * (TM / 32);
    const __amdgpu_buffer_rsrc_t xr =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.x), 0, (a.tiles_n / a.tiles_xy) * a.Cin * HW * 4, 0x00020000);
    const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.wp), 0, 9 * blocks * Mf * kSplitFragBytes, 0x00020000);
    u32x4* const patches = reinterpret_cast<u32x4*>(smem);           // BUFFERS of them, of the blocks in turn

    // this thread's fill items: (pixel of the patch, channels 8 j .. 8 j + 7 of the block)
    unsigned goff[ITEMS];
    int loff[ITEMS];
#pragma unroll
    for (int t = 0; t < ITEMS; ++t) {
        const int idx = tid + kBlock * t;
        const int j = idx >= P ? 1 : 0, pixel = idx - (idx >= P ? P : 0);
        const int pr = (pixel + skip) / Wp, pc = pixel + skip - pr * Wp;
        const int iy = iy_a + pr, ix = ix_a + pc;
        const bool item = live && idx < 2 * P;
        const bool inside = item && (unsigned)iy < (unsigned)a.H && (unsigned)ix < (unsigned)a.W;
        goff[t] = inside ? (unsigned)(((img * a.Cin + 8 * j) * HW + iy * a.W + ix) * 4) : kOutside;
        loff[t] = item ? 2 * pixel + (j ^ ((pixel >> 2) & 1)) : -1;     // in units of 16 bytes
    }
    // the patch pixel under tap 0 of this lane's output pixels
    int base[PX];
#pragma unroll
    for (int jn = 0; jn < PX; ++jn) {
        const int px = p0 + min(n[jn] * 32 + r, npx - 1);
        const int oy = px / ws, ox = px - oy * ws;
        base[jn] = (oy - oy_a) * a.stride * Wp + ox * a.stride - skip;
    }

    f32x16 high[UNITS], low[UNITS];
#pragma unroll
    for (int u = 0; u < UNITS; ++u)
#pragma unroll
        for (int q = 0; q < 16; ++q) high[u][q] = 0.f, low[u][q] = 0.f;

    float pv[ITEMS][8];
    // Loads are issued unconditionally and in a fixed order (idle items read "outside"): the compiler then counts
    // exactly how many younger loads may stay in flight at each wait.
    auto fill_load = [&](int block) {
#pragma unroll
        for (int t = 0; t < ITEMS; ++t)
#pragma unroll
            for (int q = 0; q < 8; ++q)
                pv[t][q] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xr, goff[t], (unsigned)((block * 16 + q) * HW * 4), kIn));
    };
    auto fill_store = [&](int block) {
#pragma unroll
        for (int t = 0; t < ITEMS; ++t) {
            u32x4 part[3];
            split8(pv[t], part);
            if (loff[t] >= 0) {
                u32x4* s = patches + block % BUFFERS * 3 * PLANE + loff[t];
                s[0] = part[0], s[PLANE] = part[1], s[2 * PLANE] = part[2];
            }
        }
    };
    u32x4 af[ST][FM][3], am[FM][3];
    auto a_load = [&](u32x4 (&to)[3], int i, int block, int tap) {
        const FragmentOffset at = split_fragment(block * 9 + tap, 9 * blocks, by * (TM / 32) + (i == 0 ? top : 1), Mf);
#pragma unroll
        for (int p = 0; p < 3; ++p) to[p] = __builtin_amdgcn_raw_buffer_load_b128(wr, at.lane + lane * 16, at.scalar + (unsigned)(p * 1024), 0);
    };
    u32x4 bf[2][3];                                     // of the two blocks of pixels; one block: of this slice and the next one
    auto b_load = [&](int jn, int block, int tap) {
        const int pixel = base[PX == 1 ? 0 : jn] + tap / 3 * Wp + tap % 3;
        const u32x4* s = patches + block % BUFFERS * 3 * PLANE + 2 * pixel + (g ^ ((pixel >> 2) & 1));
        bf[jn][0] = s[0], bf[jn][1] = s[PLANE], bf[jn][2] = s[2 * PLANE];
    };
    // One slice (the d-th of its block): every operand is loaded again, for the next slice that needs its registers, as soon as it has
    // been used.
    auto slice = [&](u32x4 (&w)[FM][3], int d, int block, int b_tap, bool more, int a_block, int a_tap) {
        if constexpr (PX == 1) {
            if (more) b_load((d + 1) & 1, block, b_tap);
            mfma_split(w[0], bf[d & 1], high[0], low[0]);
            __builtin_amdgcn_sched_barrier(0);
            a_load(w[0], 0, a_block, a_tap);
            __builtin_amdgcn_sched_barrier(0);
            return;
        }
        mfma_split(w[0], bf[1], high[UNITS > 1], low[UNITS > 1]);
        __builtin_amdgcn_sched_barrier(0);
        if (more) b_load(1, block, b_tap);
        mfma_split(w[0], bf[0], high[0], low[0]);
        __builtin_amdgcn_sched_barrier(0);
        a_load(w[0], 0, a_block, a_tap);
        if constexpr (FM == 2) {
            mfma_split(w[1], bf[0], high[2], low[2]);
            __builtin_amdgcn_sched_barrier(0);
            a_load(w[1], 1, a_block, a_tap);
        }
        if (more) b_load(0, block, b_tap);
        __builtin_amdgcn_sched_barrier(0);
    };
    // the first of a wavefront's TAPS taps of a block; the middle tap goes to the share that has the taps before it
    auto first_tap = [&](int block) { return WK == 2 && ((kg ^ block) & 1) ? 5 : 0; };

    wait();
    if (live) {
        fill_load(0);
#pragma unroll
        for (int i = 0; i < FM; ++i) {
#pragma unroll
            for (int d = 0; d < ST; ++d) a_load(af[d][i], i, 0, first_tap(0) + d);
            if (WK == 2) a_load(am[i], i, kg, 4);
        }
        fill_store(0);
        if (BUFFERS == 2) fill_load(min(1, blocks - 1));
    }
    __syncthreads();
#pragma unroll 1                                        // unrolled twice it holds 64 registers more and runs 10 - 15 % slower
    for (int block = 0; block < blocks; ++block) {
        if (live) {
            const int t0 = first_tap(block), t1 = first_tap(block + 1);
            const bool middle = WK == 2 && t0 == 0;
            if constexpr (PX == 2) b_load(1, block, t0);
            b_load(0, block, t0);
#pragma unroll
            for (int d = 0; d < TAPS; ++d) {
                slice(af[d % ST], d, block, t0 + d + 1, d + 1 < TAPS || middle, d + ST < TAPS ? block : block + 1, d + ST < TAPS ? t0 + d + ST : t1 + d + ST - TAPS);
                if (d == (BUFFERS == 2 ? 0 : TAPS / 2)) {
                    if (BUFFERS == 2 && block + 1 < blocks) fill_store(block + 1);   // between the matrix instructions
                    fill_load(min(block + BUFFERS, blocks - 1));
                    __builtin_amdgcn_sched_barrier(0);  // keep the loads here: the compiler would sink them to their use
                }
            }
            if (middle) slice(am, TAPS, block, 0, false, block + 2, 4);
        }
        __syncthreads();                                // this block's patch has been read (and the next one's is there)
        if (BUFFERS == 1) {
            if (live && block + 1 < blocks) fill_store(block + 1);
            __syncthreads();
        }
    }
    // `count` rows of this lane in a block of 32: m0 + 8 (q / 4) + 4 g + q % 4
    auto store = [&](const f32x16& sum, int count, int m0, int cl) {
        if (cl >= npx) return;
        const int px = p0 + cl, oy = px / ws;
        const size_t at = (size_t)img * a.Cout * HWo + oy * a.Wo + x0 + px - oy * ws;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int m = m0 + 8 * (q / 4) + 4 * g + q % 4;
            if (q < count && m < a.Cout) store_with_epilogue(a.y, a.ep, at + (size_t)m * HWo, m, sum[q], fout);
        }
    };
    const int mw = by * TM + 32 * top;
    f32x16 sum[UNITS];
#pragma unroll
    for (int u = 0; u < UNITS; ++u) sum[u] = split_sum(high[u], low[u]);
    if constexpr (WK == 1) {
        if (!live) return;
        store(sum[0], 16, mw, n[0] * 32 + r);
        if constexpr (PX == 2) store(sum[1], 16, mw, n[1] * 32 + r);
    } else {
        // The two shares of K meet: the wavefronts of the first finish pixels n[0], those of the second n[1] (of the middle rows
        // one half each); what the other one finishes is handed over in LDS.
        constexpr int GIVEN = 16 + 8 * (FM - 1);
        float* const given = smem + (wave * GIVEN) * 64 + lane;
        const float* const taken = smem + ((wave ^ 2) * GIVEN) * 64 + lane;
        if (live) {
#pragma unroll
            for (int q = 0; q < 16; ++q) given[q * 64] = kg ? sum[0][q] : sum[1][q];
            if constexpr (FM == 2) {
#pragma unroll
                for (int q = 0; q < 8; ++q) given[(16 + q) * 64] = kg ? sum[2][q] : sum[2][8 + q];
            }
        }
        __syncthreads();
        if (live) {
#pragma unroll
            for (int q = 0; q < 16; ++q) sum[0][q] = (kg ? sum[1][q] : sum[0][q]) + taken[q * 64];
            if constexpr (FM == 2) {
#pragma unroll
                for (int q = 0; q < 8; ++q) sum[2][q] = (kg ? sum[2][8 + q] : sum[2][q]) + taken[(16 + q) * 64];
            }
        }
        __syncthreads();                                // the next tile's patches go here
        if (!live) return;
        store(sum[0], 16, mw, (kg ? n[1] : n[0]) * 32 + r);
        if constexpr (FM == 2) store(sum[2], 8, by * TM + 32 + 16 * kg, n[0] * 32 + r);
    }
}

// ------------------------------------------------------------------------------------
// The same for few output pixels (a batch of small maps, one image): a tile is 32 output channels by a run of 32 pixels, and K is
// split over the four wavefronts - wavefront w takes blocks w, w + 4, .. of 16 channels. Each keeps the patch of its block in
// its own quarter of the LDS (up to PM pixels), so there is no workgroup barrier until the four sums meet there at the end,
// and fetches its next block while it multiplies. The 16 x 16 tiles that gather their operands from memory spend a round
// trip per chunk of K and fetch every input nine times: alone, us, gathered and this: 14 x 14 192 -> 192, six images
// 31 -> 10, 6 x 6 384 -> 768, six images 46 -> 21, 17 x 17 192 -> 192, one image 11.5 -> 9.2.
// Needs Cin % 16 == 0 and patches of at most PM pixels.
// ------------------------------------------------------------------------------------
template <int PM, bool FIN, class Wait>
__device__ __forceinline__ void conv3x3_split_k_tile(const C3Args& a, int tile, float* smem, int tid, bool live, Wait& wait) {
    const bool fout = wait.far_out();
    constexpr int ITEMS = (2 * PM + 63) / 64, PLANE = 2 * PM, ST = 3;    // PLANE: one part of a patch, in units of 16 bytes
    constexpr int kIn = FIN ? kPolicyDeviceScope : 0;
    static_assert(4 * PM * 24 == smem_floats(KID_C3_SK) && PM * 24 >= 16 * 64, "LDS budget: four patches; a quarter holds a wavefront's sums");
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 31, g = lane >> 5;
    const int by = tile % a.co_groups, bt = tile / a.co_groups;
    const int img = bt / a.tiles_xy, seg = bt - img * a.tiles_xy;
    const int HWo = a.Ho * a.Wo, HW = a.H * a.W;
    const int p0 = seg * 32, npx = min(32, HWo - p0);
    const int oy_a = p0 / a.Wo, oy_b = (p0 + npx - 1) / a.Wo;
    const int iy_a = oy_a * a.stride - a.pad, Wp = a.W + 2 * a.pad, P = ((oy_b - oy_a) * a.stride + 3) * Wp;
    const int blocks = a.groups / 16, Mf = a.co_groups;
    const __amdgpu_buffer_rsrc_t xr =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.x), 0, (a.tiles_n / a.tiles_xy) * a.Cin * HW * 4, 0x00020000);
    const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.wp), 0, 9 * blocks * Mf * kSplitFragBytes, 0x00020000);
    u32x4* const patch = reinterpret_cast<u32x4*>(smem) + wave * 3 * PLANE;

    // this lane's fill items: (pixel of the patch, channels 8 j .. 8 j + 7 of the block)
    unsigned goff[ITEMS];
    int loff[ITEMS];
#pragma unroll
    for (int t = 0; t < ITEMS; ++t) {
        const int idx = lane + 64 * t;
        const int j = idx >= P ? 1 : 0, pixel = idx - (idx >= P ? P : 0);
        const int pr = pixel / Wp, pc = pixel - pr * Wp;
        const int iy = iy_a + pr, ix = pc - a.pad;
        const bool item = live && idx < 2 * P;
        const bool inside = item && (unsigned)iy < (unsigned)a.H && (unsigned)ix < (unsigned)a.W;
        goff[t] = inside ? (unsigned)(((img * a.Cin + 8 * j) * HW + iy * a.W + ix) * 4) : kOutside;
        loff[t] = item ? 2 * pixel + (j ^ ((pixel >> 2) & 1)) : -1;     // in units of 16 bytes
    }
    const int px = p0 + min(r, npx - 1), oy = px / a.Wo, ox = px - oy * a.Wo;
    const int base = (oy - oy_a) * a.stride * Wp + ox * a.stride;      // the patch pixel under tap 0 of this lane's pixel

    f32x16 high, low;
#pragma unroll
    for (int q = 0; q < 16; ++q) high[q] = 0.f, low[q] = 0.f;
    float pv[ITEMS][8];
    auto fill_load = [&](int block) {                   // items that few patches need are skipped by all lanes together
#pragma unroll
        for (int t = 0; t < ITEMS; ++t) {
            if (64 * t >= 2 * P) break;
#pragma unroll
            for (int q = 0; q < 8; ++q)
                pv[t][q] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xr, goff[t], (unsigned)((block * 16 + q) * HW * 4), kIn));
        }
    };
    auto fill_store = [&]() {
#pragma unroll
        for (int t = 0; t < ITEMS; ++t) {
            if (64 * t >= 2 * P) break;
            u32x4 part[3];
            split8(pv[t], part);
            if (loff[t] >= 0) patch[loff[t]] = part[0], patch[PLANE + loff[t]] = part[1], patch[2 * PLANE + loff[t]] = part[2];
        }
    };
    u32x4 af[ST][3];
    auto a_load = [&](int block, int tap, int stage) {
        const FragmentOffset at = split_fragment(block * 9 + tap, 9 * blocks, by, Mf);
#pragma unroll
        for (int p = 0; p < 3; ++p) af[stage][p] = __builtin_amdgcn_raw_buffer_load_b128(wr, at.lane + lane * 16, at.scalar + (unsigned)(p * 1024), 0);
    };
    auto b_load = [&](u32x4 (&bf)[3], int tap) {
        const int pixel = base + (tap / 3) * Wp + tap % 3;
        const u32x4* s = patch + 2 * pixel + (g ^ ((pixel >> 2) & 1));
        bf[0] = s[0], bf[1] = s[PLANE], bf[2] = s[2 * PLANE];
    };
    // Lanes of one wavefront exchange the patch through LDS: its LDS operations are carried out in order, the fence keeps the
    // compiler from reordering them.
    auto wave_fence = [] {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };

    if (live && wave < blocks) {
#pragma unroll
        for (int d = 0; d < ST; ++d) a_load(wave, d, d);
    }
    wait();
    if (live && wave < blocks) {
        fill_load(wave);
#pragma unroll 1
        for (int block = wave; block < blocks; block += 4) {
            wave_fence();                               // the previous block's patch has been read
            fill_store();
            wave_fence();
            if (block + 4 < blocks) fill_load(block + 4);
            __builtin_amdgcn_sched_barrier(0);          // keep the loads here: the compiler would sink them to their use
            u32x4 bf[2][3];
            b_load(bf[0], 0);
#pragma unroll
            for (int tap = 0; tap < 9; ++tap) {
                if (tap < 8) b_load(bf[(tap + 1) & 1], tap + 1);   // next tap's B fragments, before this tap's matrix instructions
                mfma_split(af[tap % ST], bf[tap & 1], high, low);
                a_load(tap + ST < 9 ? block : block + 4, (tap + ST) % 9, tap % ST);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    // the four sums meet: each wavefront leaves its own where its patch was and adds up four rows of every eight
    const f32x16 own = split_sum(high, low);
    wave_fence();
    float* const sums = smem + wave * 3 * PLANE * 4;
    if (live) {
#pragma unroll
        for (int q = 0; q < 16; ++q) sums[q * 64 + lane] = own[q];
    }
    __syncthreads();
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    if (live) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int w = 0; w < 4; ++w) v[q] += smem[w * 3 * PLANE * 4 + (4 * wave + q) * 64 + lane];
    }
    __syncthreads();                                    // the next tile's patches go here
    if (!live || r >= npx) return;
    const int mw = by * 32 + 8 * wave + 4 * g;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int m = mw + q;
        if (m < a.Cout) store_with_epilogue(a.y, a.ep, ((size_t)img * a.Cout + m) * HWo + p0 + r, m, v[q], fout);
    }
}

// ------------------------------------------------------------------------------------
// conv1x1 / fc for many output pixels on the plan of the patch-stationary conv3x3: Y[Cout x cols] = W[Cout x Cin] X[Cin x cols],
// tile = TM output channels x 64 consecutive columns (a run may cross from one image into the next), in split bf16. KB blocks of
// 16 input channels of the tile's columns sit in LDS, split into three parts (32 bytes per column and part, as above), in two
// buffers: while one is multiplied, the next is split into the other and the loads of the one after that are in flight - one
// barrier per KB blocks. The weights ([Cin / 16][CoutP / 32][part][lane][8]) go from memory straight into operands, one
// chunk ahead. ROWS = 64: 2 x 2 wavefronts of 32 x 32 outputs. ROWS = 32 (fewer than 200 tiles of 64 x 64): 1 x 2, and the
// other two wavefronts take every second block of 16 channels; the halves of the sums meet in LDS at the end.
// Splitting the activations (5.5 vector instructions per element for 64 rows) and the vector L1 bound it: 17 x 17 768 -> 192 at
// batch 32 35 -> 28 us, 8 x 8 2048 -> 320 49 -> 39 us with the fp32 matrix instructions and with these.
// Needs Cin % 16 == 0.
// ------------------------------------------------------------------------------------
template <int ROWS, int KB, bool FIN, class Wait>
__device__ __forceinline__ void conv1x1_patch_tile(const PwArgs& a, int tile, float* smem, int tid, bool live, Wait& wait) {
    const bool fout = wait.far_out();
    constexpr int TM = ROWS, TN = 64, KW = ROWS == 32 ? 2 : 1, OWN = KB / KW;
    constexpr int PLANE = 2 * TN, BUFFER = KB * 3 * PLANE, ITEMS = KB / 2;                // LDS in units of 16 bytes
    constexpr int kIn = FIN ? kPolicyDeviceScope : 0;
    static_assert(2 * BUFFER * 4 <= (KB == 2 ? kSmemFloatsPatch : 2 * kSmemFloatsPatch) && KB % 2 == 0 && TN * 4 == kBlock && (ROWS == 32 || ROWS == 64), "LDS budget");
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = ROWS == 32 ? wave >> 1 : 0, wm = ROWS == 32 ? 0 : wave >> 1, wn = wave & 1, r = lane & 31, g = lane >> 5;
    const int by = tile % a.mtiles, bx = tile / a.mtiles;
    const int mw = by * TM + wm * 32, n0 = bx * TN;
    const int blocks = a.ksteps / 16, chunks = (blocks + KB - 1) / KB, Mf = a.mtiles * (TM / 32);
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.x), 0, a.cols * a.Cin * 4, 0x00020000);
    const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.wp), 0, blocks * Mf * kSplitFragBytes, 0x00020000);
    // this thread's fill items: column c of the tile, channels 8 j .. 8 j + 7 of blocks b0, b0 + 2, .. of a chunk
    const int c = tid % TN, j = (tid / TN) & 1, b0 = tid / (2 * TN);
    unsigned goff;
    {
        const int col = n0 + c;
        const int img = col / a.HW, pix = col - img * a.HW;
        goff = (live && col < a.cols) ? (unsigned)(((img * a.Cin + 8 * j) * a.HW + pix) * 4) : kOutside;
    }
    const int loff = b0 * 3 * PLANE + 2 * c + (j ^ ((c >> 2) & 1));
    const int cl = wn * 32 + r, lbase = 2 * cl + (g ^ ((cl >> 2) & 1));

    f32x16 high, low;
#pragma unroll
    for (int q = 0; q < 16; ++q) high[q] = 0.f, low[q] = 0.f;

    float pv[ITEMS][8];
    // loads are issued unconditionally and in a fixed order (blocks beyond Cin read "outside"): the compiler then counts
    // exactly how many younger loads may stay in flight at each wait
    auto fill_load = [&](int chunk) {
#pragma unroll
        for (int t = 0; t < ITEMS; ++t) {
            const int block = chunk * KB + b0 + 2 * t;
            const unsigned off = goff != kOutside && block < blocks ? goff + (unsigned)(block * 16 * a.HW * 4) : kOutside;
#pragma unroll
            for (int q = 0; q < 8; ++q) pv[t][q] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xr, off, (unsigned)(q * a.HW * 4), kIn));
        }
    };
    u32x4* const lds = reinterpret_cast<u32x4*>(smem);
    auto fill_store = [&](int buffer) {
#pragma unroll
        for (int t = 0; t < ITEMS; ++t) {
            u32x4 part[3];
            split8(pv[t], part);
            u32x4* s = lds + buffer * BUFFER + loff + t * 6 * PLANE;
            s[0] = part[0], s[PLANE] = part[1], s[2 * PLANE] = part[2];
        }
    };
    u32x4 af[OWN][3];
    auto a_load = [&](int chunk, int own) {             // a block beyond Cin: zeros
        const FragmentOffset at = split_fragment(chunk * KB + own * KW + kg, blocks, mw / 32, Mf);
#pragma unroll
        for (int p = 0; p < 3; ++p) af[own][p] = __builtin_amdgcn_raw_buffer_load_b128(wr, at.lane + lane * 16, at.scalar + (unsigned)(p * 1024), 0);
    };

    wait();
    if (live) {
        fill_load(0);
#pragma unroll
        for (int own = 0; own < OWN; ++own) a_load(0, own);
        fill_store(0);
        fill_load(1);
    }
    __syncthreads();
#pragma unroll 1
    for (int chunk = 0; chunk < chunks; ++chunk) {
        if (live) {
            const u32x4* s0 = lds + (chunk & 1) * BUFFER + kg * 3 * PLANE + lbase;
#pragma unroll
            for (int own = 0; own < OWN; ++own) {
                u32x4 bf[3];
#pragma unroll
                for (int p = 0; p < 3; ++p) bf[p] = s0[(own * KW * 3 + p) * PLANE];
                mfma_split(af[own], bf, high, low);
                a_load(chunk + 1, own);
            }
            if (chunk + 1 < chunks) fill_store((chunk + 1) & 1);
            fill_load(chunk + 2);
        }
        __syncthreads();                                // the chunk is used up, the next one is there
    }
    f32x16 sum = split_sum(high, low);
    if (KW > 1) {                                       // the second half of K joins the first
        if (kg == 1) {
#pragma unroll
            for (int q = 0; q < 16; ++q) smem[(wn * 16 + q) * 64 + lane] = sum[q];
        }
        __syncthreads();
        if (kg == 0) {
#pragma unroll
            for (int q = 0; q < 16; ++q) sum[q] += smem[(wn * 16 + q) * 64 + lane];
        }
        __syncthreads();                                // the next tile writes here
    }
    const int col = n0 + cl;
    if (!live || kg != 0 || col >= a.cols) return;
    const int img = col / a.HW, pix = col - img * a.HW;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int m = mw + 8 * (q / 4) + 4 * g + q % 4;
        if (m < a.Cout)
            store_with_epilogue(a.y, a.ep, ((size_t)img * a.Cout + m) * a.HW + pix, m, sum[q] + (a.bias ? a.bias[m] : 0.f), fout);
    }
}

// ------------------------------------------------------------------------------------
// conv1x1 for small problems (the batch-1 case): latency, not throughput, decides.
// A workgroup owns a 32 x 32 output tile as 2 x 2 MFMA tiles; its four wavefronts split K
// four ways, each accumulates all four MFMA tiles over its quarter of K with operands
// loaded straight from global memory into registers - no LDS staging and no barrier in
// the K loop, up to 64 loads in flight per lane - and the four partial results are summed
// through LDS in a fixed order (wavefront 0 + 1 + 2 + 3), so the result does not depend
// on timing. The weights are read from a copy repacked once, ahead of time, into the order
// the A operand wants: block (row tile rt, k step ks) holds W[16 rt + l % 16][4 ks + l / 16]
// for lane l = 0..63, zero outside the matrix, so one A load is one contiguous 256 bytes.
// The copy is zero-padded along K to a multiple of 4 x chunk steps: every wavefront runs
// whole chunks and the K loop needs no tail handling (a lone wavefront per SIMD issues one
// instruction every few cycles, so instruction count is what these kernels pay for).
// ------------------------------------------------------------------------------------
template <int CH, bool FIN, class Wait>          // CH k steps per chunk: 4 * CH loads in flight per lane
__device__ __forceinline__ void conv1x1_direct_tile(const PwArgs& a, int tile, float* smem, int tid, bool live, Wait& wait) {
    const bool fout = wait.far_out();       // device-scope stores: some reader of the result sits on another XCD
    wait();
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int by = tile / a.tiles_n, bx = tile - by * a.tiles_n;
    const int m0 = by * 32, n0 = bx * 32;
    const int S = a.ksteps;                                  // padded: every wavefront owns S / 4 steps, a multiple of CH
    const int steps = S >> 2;
    const unsigned k_last = (unsigned)(a.Cin - 1) * (unsigned)a.HW;   // offset of the last real input row
    const unsigned k_step = 4u * (unsigned)a.HW;

    const float* ap[2];
    const float* xb[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int rt = min(by * 2 + i, a.mtiles - 1);       // a row tile past the matrix repeats the last one; never stored
        ap[i] = a.wp + ((size_t)rt * S + (size_t)wave * steps) * 64 + lane;
        const int col = min(n0 + i * 16 + (lane & 15), a.cols - 1);
        const int img = col / a.HW, pix = col - img * a.HW;
        xb[i] = a.x + (size_t)img * a.Cin * a.HW + pix;
    }
    // offset of this lane's input row at the wavefront's first step; rows past Cin (zero
    // weights there) are clamped onto the last real row so that every load stays in bounds
    unsigned koff = (unsigned)(4 * wave * steps + (lane >> 4)) * (unsigned)a.HW;
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    for (int s0 = 0; s0 < (live ? steps : 0); s0 += CH) {
        float av[2][CH], bv[2][CH];
#pragma unroll
        for (int q = 0; q < CH; ++q) {
            const unsigned off = min(koff + (unsigned)q * k_step, k_last);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                av[i][q] = ap[i][q * 64];
                bv[i][q] = ldg(a.x, xb[i] + off, FIN);
            }
        }
        __builtin_amdgcn_sched_barrier(0);                   // every load of the chunk is issued before the first use
#pragma unroll
        for (int q = 0; q < CH; ++q)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i][q], bv[j][q], acc[i][j], 0, 0, 0);
        ap[0] += CH * 64, ap[1] += CH * 64;
        koff += CH * k_step;
    }
    // partial sums -> LDS as red[wave][tile][reg][lane]; wavefront w then finishes MFMA tile w
    static_assert(4 * 4 * 4 * 64 <= kSmemFloats, "LDS budget");
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) smem[((wave * 4 + i * 2 + j) * 4 + r) * 64 + lane] = acc[i][j][r];
    __syncthreads();
    {
        const int ti = wave >> 1, tj = wave & 1;
        const int col = n0 + tj * 16 + (lane & 15);
        const int ccol = min(col, a.cols - 1);
        const int img = ccol / a.HW, pix = ccol - img * a.HW;
        float* yb = a.y + (size_t)img * a.Cout * a.HW + pix;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float sum = smem[((0 * 4 + wave) * 4 + r) * 64 + lane];
#pragma unroll
            for (int w2 = 1; w2 < 4; ++w2) sum += smem[((w2 * 4 + wave) * 4 + r) * 64 + lane];
            const int m = m0 + ti * 16 + 4 * (lane >> 4) + r;
            if (m < a.Cout && col < a.cols && live) {
                const float b = a.bias ? a.bias[m] : 0.f;
                store_with_epilogue(a.y, a.ep, (size_t)(yb - a.y) + (size_t)m * a.HW, m, sum + b, fout);
            }
        }
    }
    __syncthreads();                                         // LDS is reused by the next tile
}

// ------------------------------------------------------------------------------------
// conv1x1 for the smallest problems (one image, a few thousand pixels at most), where the
// time goes into issuing loads and into waiting, not into arithmetic. Differences from the
// 32 x 32 kernel above:
//   * the output tile is 16 channels wide only, so a problem spreads over as many compute
//     units as possible (an fp32 MFMA occupies its SIMD for 32 cycles: few tiles means
//     few SIMDs working);
//   * the packed weights hold 4 k-steps per lane (block (row tile, group g), lane l, word q
//     = W[16 rt + l % 16][16 g + 4 q + l / 16]): one 128-bit load feeds 4 MFMAs;
//   * VEC (pixels per plane a multiple of 4): activations are read 128 bits at a time. Lane l
//     loads X[k][n0 + 4 (l % 16) .. + 3]; word j of that load is the B operand of MFMA tile j,
//     whose columns are n0 + 4 i + j, i = 0..15 - four interleaved 16-column tiles, 64 columns
//     per workgroup, and the four results of a lane are again 4 consecutive pixels: one
//     128-bit store;
//   * otherwise the tile is 16 x 16 and activations are read word by word.
// K is split over the four wavefronts in groups of 4 k-steps, G groups in flight at a time;
// partial sums are added through LDS in a fixed order.
// ------------------------------------------------------------------------------------
template <int G, bool VEC, bool EA, bool FIN, class Wait>
__device__ __forceinline__ void conv1x1_k4_tile(const typename std::conditional<EA, PwAddArgs, PwArgs>::type& a, int tile, float* smem,
                                                int tid, bool live, Wait& wait) {
    const bool fout = wait.far_out();       // device-scope stores: some reader of the result sits on another XCD
    constexpr int NJ = VEC ? 4 : 1;                          // MFMA tiles per wavefront
    constexpr int TN = VEC ? 64 : 16;                        // columns per workgroup tile
    static_assert(4 * NJ * 4 * 64 <= kSmemFloats, "LDS budget");
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int by = tile / a.tiles_n, bx = tile - by * a.tiles_n;
    const int colv = bx * TN + (VEC ? 4 : 1) * (lane & 15);  // first column this lane owns
    // addresses first (nothing is read yet), then the wait for the producers
    const int groups = a.ksteps;                             // groups of 4 k-steps in the packed copy, a multiple of 4 G
    const int gw = groups >> 2;                              // groups per wavefront
    const f32x4* ap = reinterpret_cast<const f32x4*>(a.wp) + ((size_t)by * groups + (size_t)wave * gw) * 64 + lane;
    const int col = min(colv, a.cols - (VEC ? 4 : 1));       // columns past the end repeat the last ones; never stored
    const int img = col / a.HW, pix = col - img * a.HW;
    const float* xb = a.x + (size_t)img * a.Cin * a.HW + pix;
    const unsigned k_last = (unsigned)(a.Cin - 1) * (unsigned)a.HW;       // rows past Cin (zero weights) repeat the last row
    const unsigned k_step = 4u * (unsigned)a.HW;
    unsigned koff = (unsigned)(16 * wave * gw + (lane >> 4)) * (unsigned)a.HW;
    // wavefront w finishes accumulator register w of every MFMA tile: output row 4 (lane / 16) + w
    const int m = by * 16 + 4 * (lane >> 4) + wave;
    float es = 1.f, et = 0.f;
    if (a.ep.y != nullptr && a.ep.scale != nullptr) es = a.ep.scale[min(m, a.Cout - 1)], et = a.ep.shift[min(m, a.Cout - 1)];
    wait();
    if (live) {
        f32x4 acc[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int g0 = 0; g0 < gw; g0 += G) {
            f32x4 av[G];
            float bv[G][4][NJ];
#pragma unroll
            for (int gi = 0; gi < G; ++gi) {
                av[gi] = ap[gi * 64];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const unsigned off = min(koff + (unsigned)(4 * gi + q) * k_step, k_last);
                    if (VEC) {
                        const float4 v = ldg4(a.x, xb + off, FIN);
                        __builtin_memcpy(bv[gi][q], &v, sizeof v);
                    } else {
                        bv[gi][q][0] = ldg(a.x, xb + off, FIN);
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);               // every load of the chunk is issued before the first use
#pragma unroll
            for (int gi = 0; gi < G; ++gi)
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int j = 0; j < NJ; ++j)
                        acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[gi][q], bv[gi][q][j], acc[j], 0, 0, 0);
            ap += G * 64;
            koff += 4u * G * k_step;
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) smem[((wave * NJ + j) * 4 + r) * 64 + lane] = acc[j][r];
    }
    __syncthreads();
    bool valid = false;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    size_t at = 0;
    if (live) {
        float out[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            float sum = smem[((0 * NJ + j) * 4 + wave) * 64 + lane];
#pragma unroll
            for (int w2 = 1; w2 < 4; ++w2) sum += smem[((w2 * NJ + j) * 4 + wave) * 64 + lane];
            out[j] = sum;
        }
        valid = m < a.Cout && colv < a.cols;                 // VEC: cols is a multiple of 4, a lane's 4 columns are all in or all out
        if (valid) {
            const float b = a.bias ? a.bias[m] : 0.f;
            const int img = colv / a.HW, pix = colv - img * a.HW;
            at = ((size_t)img * a.Cout + m) * a.HW + pix;
            v = make_float4(out[0] + b, out[NJ > 1 ? 1 : 0] + b, out[NJ > 2 ? 2 : 0] + b, out[NJ > 3 ? 3 : 0] + b);
            if (VEC) stg4(a.y, a.y + at, v, fout);
            else stg(a.y, a.y + at, v.x, fout);
            if (a.ep.y != nullptr) {
                v.x = fmaf(v.x, es, et), v.y = fmaf(v.y, es, et), v.z = fmaf(v.z, es, et), v.w = fmaf(v.w, es, et);
                if (a.ep.relu) v.x = fmaxf(v.x, 0.f), v.y = fmaxf(v.y, 0.f), v.z = fmaxf(v.z, 0.f), v.w = fmaxf(v.w, 0.f);
                if (VEC) stg4(a.ep.y, a.ep.y + at, v, fout);
                else stg(a.ep.y, a.ep.y + at, v.x, fout);
            }
        }
    }
    if constexpr (EA) {
        wait.late();
        if (valid) add_epilogue<VEC>(a.ea, v, at, fout);
    }
    __syncthreads();                                         // LDS is reused by the next tile
}

// ------------------------------------------------------------------------------------
// conv3x3 dense on the vector ALUs: one thread = one output pixel x 8 output channels.
// Input patches go through LDS (4 input channels per slice); the weights a wavefront
// needs are the same for all of its lanes, so they are read through uniform addresses.
// TP = 16: the workgroup owns a 16 x 16 pixel tile and one group of 8 output channels.
// TP = 8 : each wavefront owns the same 8 x 8 pixel tile and its own group of 8 channels.
// Tile index = (image * co_groups + channel group) * tiles_xy + pixel tile.
// ------------------------------------------------------------------------------------
template <int TP, int S, bool FIN, class Wait>
__device__ __forceinline__ void conv3x3_tile(const C3Args& a, int tile, float* smem, int tid, bool live, Wait& wait) {
    const bool fout = wait.far_out();       // device-scope stores: some reader of the result sits on another XCD
    wait();
    constexpr int CIC = S == 2 && TP == 16 ? 2 : 4;    // input channels per LDS slice
    constexpr int IW = (TP - 1) * S + 3;               // input patch edge
    constexpr int LDP = IW + 1;
    constexpr int GROUPS = TP == 16 ? 1 : 4;           // channel groups per workgroup
    constexpr int CO = 8;
    constexpr int WROW = 12;                           // a (channel, input channel) pair's nine taps, padded to three 128-bit reads
    constexpr int NW = GROUPS * CO * CIC;              // such pairs per slice
    static_assert(CIC * IW * LDP + NW * WROW <= kSmemFloats && (CIC * IW * LDP) % 4 == 0, "LDS budget; the weights start 16-byte aligned");
    float* patch = smem;                               // [CIC][IW][LDP]
    float* wsm = smem + CIC * IW * LDP;                // [GROUPS CO][CIC][WROW]: the slice's weights of every output channel of the workgroup

    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int local = TP == 16 ? tid : (tid & 63);
    const int ty = local / TP, tx = local % TP;
    const int ptile = tile % a.tiles_xy, rest = tile / a.tiles_xy;
    const int cog = rest % a.co_groups, img = rest / a.co_groups;
    const int tile_y = ptile / a.tiles_x, tile_x = ptile - tile_y * a.tiles_x;
    const int oy = tile_y * TP + ty, ox = tile_x * TP + tx;
    const int co0 = (cog * GROUPS + (TP == 16 ? 0 : wave)) * CO;
    const int iy0 = tile_y * TP * S - a.pad, ix0 = tile_x * TP * S - a.pad;
    const float* xin = a.x + (size_t)img * a.Cin * a.H * a.W;

    float acc[CO];
#pragma unroll
    for (int j = 0; j < CO; ++j) acc[j] = 0.f;
    // The weights go through LDS with the patch (one batch of loads, one barrier): read through uniform addresses
    // straight from memory they arrived a few at a time, each batch a trip to L2 that the wavefront waited for, and
    // that, not arithmetic or bandwidth, was the tile's 8 us on a stem. Out-of-range channels repeat the last one and are
    // masked at the store.
    const int cbase = cog * GROUPS * CO;               // first output channel of the workgroup
    const int wgroup = TP == 16 ? 0 : wave;

    for (int c0 = 0; c0 < a.Cin; c0 += CIC) {
        if (live) {
            constexpr int NL = (CIC * IW * IW + kBlock - 1) / kBlock;   // loads per thread, all in flight
            float pv[NL];
#pragma unroll
            for (int q = 0; q < NL; ++q) {
                const int e = min(tid + q * kBlock, CIC * IW * IW - 1);
                const int cx = e % IW, t = e / IW;
                const int cy = t % IW, ci = t / IW;
                const int gy = iy0 + cy, gx = ix0 + cx, gc = c0 + ci;
                const bool in = gc < a.Cin && gy >= 0 && gy < a.H && gx >= 0 && gx < a.W;
                const float v = ldg(a.x, xin + ((size_t)min(gc, a.Cin - 1) * a.H + min(max(gy, 0), a.H - 1)) * a.W + min(max(gx, 0), a.W - 1), FIN);
                pv[q] = in ? v : 0.f;
            }
            constexpr int NWL = (NW * 9 + kBlock - 1) / kBlock;         // weight loads per thread
            float wv[NWL];
#pragma unroll
            for (int q = 0; q < NWL; ++q) {
                const int e = min(tid + q * kBlock, NW * 9 - 1);
                const int tap = e % 9, pair = e / 9, ci = pair % CIC, jj = pair / CIC;
                const float v = a.w[((size_t)min(cbase + jj, a.Cout - 1) * a.Cin + min(c0 + ci, a.Cin - 1)) * 9 + tap];
                wv[q] = c0 + ci < a.Cin ? v : 0.f;
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < NL; ++q) {
                const int e = tid + q * kBlock;
                if (e < CIC * IW * IW) {
                    const int cx = e % IW, t = e / IW;
                    const int cy = t % IW, ci = t / IW;
                    patch[(ci * IW + cy) * LDP + cx] = pv[q];
                }
            }
#pragma unroll
            for (int q = 0; q < NWL; ++q) {
                const int e = tid + q * kBlock;
                if (e < NW * 9) wsm[(e / 9) * WROW + e % 9] = wv[q];
            }
        }
        __syncthreads();
        const int nci = live ? min(CIC, a.Cin - c0) : 0;
        for (int ci = 0; ci < nci; ++ci) {
            float in[9];
#pragma unroll
            for (int dr = 0; dr < 3; ++dr)
#pragma unroll
                for (int dc = 0; dc < 3; ++dc) in[dr * 3 + dc] = patch[(ci * IW + ty * S + dr) * LDP + tx * S + dc];
#pragma unroll
            for (int j = 0; j < CO; ++j) {
                const float4* wp = reinterpret_cast<const float4*>(wsm + ((wgroup * CO + j) * CIC + ci) * WROW);   // the same address in every lane: a broadcast
                const float4 w0 = wp[0], w1 = wp[1], w2 = wp[2];
                const float wq[9] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w, w2.x};
#pragma unroll
                for (int q = 0; q < 9; ++q) acc[j] = fmaf(wq[q], in[q], acc[j]);
            }
        }
        __syncthreads();
    }
    if (oy < a.Ho && ox < a.Wo && live) {
#pragma unroll
        for (int j = 0; j < CO; ++j)
            if (co0 + j < a.Cout)
                store_with_epilogue(a.y, a.ep, (((size_t)img * a.Cout + co0 + j) * a.Ho + oy) * a.Wo + ox, co0 + j, acc[j], fout);
    }
}

// ------------------------------------------------------------------------------------
// conv3x3 as an implicit GEMM on the matrix cores: Y[Cout x cols] = W[Cout x 9 Cin] * P[9 Cin x cols]
// with cols = N * Ho * Wo and P[(ci, dr, dc)][(n, oy, ox)] = x[n][ci][oy S - pad + dr][ox S - pad + dc]
// (zero outside the image), gathered straight from global memory: the weight tensor
// [Cout][Cin][3][3] already is that W, row-major, so it is repacked exactly like a 1x1
// weight matrix with 9 Cin input channels. Same structure as the 16 x 16 conv1x1 above: K split
// over the four wavefronts in groups of 4 k-steps, G groups in flight, fixed-order reduction.
// A lane walks k in steps of 4, so (ci, tap) is updated incrementally: tap += 4, carry into ci.
// ------------------------------------------------------------------------------------
template <int G, bool EA, bool FIN, class Wait>
__device__ __forceinline__ void conv3x3_k4_tile(const typename std::conditional<EA, C3AddArgs, C3Args>::type& a, int tile, float* smem,
                                                int tid, bool live, Wait& wait) {
    const bool fout = wait.far_out();       // device-scope stores: some reader of the result sits on another XCD
    static_assert(4 * 4 * 64 <= kSmemFloats, "LDS budget");
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int by = tile / a.tiles_n, bx = tile - by * a.tiles_n;
    const int colv = bx * 16 + (lane & 15);
    const int HWo = a.Ho * a.Wo;
    // addresses first (nothing is read yet), then the wait for the producers
    const int groups = a.groups, gw = groups >> 2;
    const f32x4* ap = reinterpret_cast<const f32x4*>(a.wp) + ((size_t)by * groups + (size_t)wave * gw) * 64 + lane;
    const int col = min(colv, a.cols - 1);                   // columns past the end repeat the last one; never stored
    const int img = col / HWo, pix = col - img * HWo;
    const int oy = pix / a.Wo, ox = pix - oy * a.Wo;
    const int iy0 = oy * a.stride - a.pad, ix0 = ox * a.stride - a.pad;
    const int HW = a.H * a.W;
    const float* xb = a.x + (size_t)img * a.Cin * HW;
    const int k0 = 16 * wave * gw + (lane >> 4);             // this lane's first k; then + 4 per k-step
    int ci = k0 / 9, tap = k0 - 9 * ci;
    const int m = by * 16 + 4 * (lane >> 4) + wave;          // wavefront w finishes accumulator register w
    float es = 1.f, et = 0.f;
    if (a.ep.y != nullptr && a.ep.scale != nullptr) es = a.ep.scale[min(m, a.Cout - 1)], et = a.ep.shift[min(m, a.Cout - 1)];
    wait();
    if (live) {
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int g0 = 0; g0 < gw; g0 += G) {
            f32x4 av[G];
            float bv[G][4];
            unsigned inside = 0;
#pragma unroll
            for (int gi = 0; gi < G; ++gi) {
                av[gi] = ap[gi * 64];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int dr = (tap * 11) >> 5, dc = tap - 3 * dr;       // tap / 3, tap % 3 for tap < 9
                    const int iy = iy0 + dr, ix = ix0 + dc;
                    const bool in = ci < a.Cin && (unsigned)iy < (unsigned)a.H && (unsigned)ix < (unsigned)a.W;
                    inside |= (in ? 1u : 0u) << (gi * 4 + q);
                    const int off = min(ci, a.Cin - 1) * HW + min(max(iy, 0), a.H - 1) * a.W + min(max(ix, 0), a.W - 1);
                    bv[gi][q] = ldg(a.x, xb + off, FIN);
                    tap += 4;
                    if (tap >= 9) tap -= 9, ++ci;
                }
            }
            __builtin_amdgcn_sched_barrier(0);               // every load of the chunk is issued before the first use
#pragma unroll
            for (int gi = 0; gi < G; ++gi)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[gi][q], ((inside >> (gi * 4 + q)) & 1u) ? bv[gi][q] : 0.f, acc, 0, 0, 0);
            ap += G * 64;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) smem[(wave * 4 + r) * 64 + lane] = acc[r];
    }
    __syncthreads();
    bool valid = false;
    float z = 0.f;
    size_t at = 0;
    if (live) {
        float sum = smem[(0 * 4 + wave) * 64 + lane];
#pragma unroll
        for (int w2 = 1; w2 < 4; ++w2) sum += smem[(w2 * 4 + wave) * 64 + lane];
        valid = m < a.Cout && colv < a.cols;
        if (valid) {
            const int img = colv / HWo, pix = colv - img * HWo;
            at = ((size_t)img * a.Cout + m) * HWo + pix;
            stg(a.y, a.y + at, sum, fout);
            z = sum;
            if (a.ep.y != nullptr) {
                z = fmaf(sum, es, et);
                if (a.ep.relu) z = fmaxf(z, 0.f);
                stg(a.ep.y, a.ep.y + at, z, fout);
            }
        }
    }
    if constexpr (EA) {
        wait.late();
        if (valid) add_epilogue<false>(a.ea, make_float4(z, 0.f, 0.f, 0.f), at, fout);
    }
    __syncthreads();                                         // LDS is reused by the next tile
}

// ------------------------------------------------------------------------------------
// pool3x3 for large tensors (batches): a thread computes 4 outputs of one output column, one below the other;
// neighbouring lanes have neighbouring columns, so every load and store of a wavefront is a contiguous run. The 3 + 3 STRIDE
// input rows x 3 columns the four windows cover are loaded once (4.5 loads per output at stride 1 instead of 9, each
// touching 2-3 cache lines per wavefront), reduced along the rows first and then down the column; row / column validity
// is worked out once per thread. Items = (plane, block of 4 output rows, output column) in that order.
// (Four neighbouring outputs of a ROW per thread was measured first and is slower than one output per thread: lanes
// 16 bytes apart make every load instruction touch eight cache lines.)
// ------------------------------------------------------------------------------------
template <int STRIDE, bool FIN, class Wait>
__device__ __forceinline__ void pool3x3_col_tile(const PoolArgs& a, int tile, float*, int tid, bool live, Wait& wait) {
    const bool fout = wait.far_out();
    constexpr int NR = 3 + 3 * STRIDE;                       // input rows under four windows one below the other
    const int blocks = (a.Ho + 3) >> 2;
    const int items = (a.total / (a.Ho * a.Wo)) * blocks * a.Wo;
    const int item = tile * kBlock + tid;
    const bool active = live && item < items;
    const int it = min(item, items - 1);
    const int ow = it % a.Wo, t1 = it / a.Wo;
    const int blk = t1 % blocks, plane = t1 / blocks;
    const int oh0 = 4 * blk, r0 = oh0 * STRIDE - a.pad, c0 = ow * STRIDE - a.pad;
    const float* src = a.x + (size_t)plane * a.H * a.W;
    wait();
    if (!active) return;
    const bool max_mode = a.mode == 0;
    const float neutral = max_mode ? -INFINITY : 0.f;
    float v[NR][3];
    bool row_in[NR], col_in[3];
#pragma unroll
    for (int dr = 0; dr < NR; ++dr) row_in[dr] = (unsigned)(r0 + dr) < (unsigned)a.H;
#pragma unroll
    for (int dc = 0; dc < 3; ++dc) col_in[dc] = (unsigned)(c0 + dc) < (unsigned)a.W;
    int cc[3];
#pragma unroll
    for (int dc = 0; dc < 3; ++dc) cc[dc] = min(max(c0 + dc, 0), a.W - 1);
#pragma unroll
    for (int dr = 0; dr < NR; ++dr) {
        const float* row = src + min(max(r0 + dr, 0), a.H - 1) * a.W;
#pragma unroll
        for (int dc = 0; dc < 3; ++dc) v[dr][dc] = ldg(a.x, row + cc[dc], FIN);
    }
    __builtin_amdgcn_sched_barrier(0);                       // all loads are issued before the first use
    float rowv[NR];                                          // along the rows: columns outside the image do not take part
#pragma unroll
    for (int dr = 0; dr < NR; ++dr) {
        float acc = neutral;
#pragma unroll
        for (int dc = 0; dc < 3; ++dc) {
            const float x = col_in[dc] ? v[dr][dc] : neutral;
            acc = max_mode ? fmaxf(acc, x) : acc + x;
        }
        rowv[dr] = row_in[dr] ? acc : neutral;
    }
    const int cols = (int)col_in[0] + (int)col_in[1] + (int)col_in[2];
    float* out = a.y + ((size_t)plane * a.Ho + oh0) * a.Wo + ow;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (oh0 + j >= a.Ho) break;
        const int b = j * STRIDE;
        float acc = max_mode ? fmaxf(fmaxf(rowv[b], rowv[b + 1]), rowv[b + 2]) : (rowv[b] + rowv[b + 1]) + rowv[b + 2];
        if (!max_mode) acc = acc / (float)(cols * ((int)row_in[b] + (int)row_in[b + 1] + (int)row_in[b + 2]));
        stg(a.y, out + (size_t)j * a.Wo, acc, fout);
    }
}

// ------------------------------------------------------------------------------------
// floor(e / d) for 0 <= e < 2^20 and 1 <= d, with rcp = 1 / d up to one unit in the last place: (e + 0.5) / d is at least 0.5 / d
// away from an integer, the rounding errors of the reciprocal and the product are below e 2^-22 / d.
__device__ __forceinline__ int small_div(int e, float rcp) { return (int)(((float)e + 0.5f) * rcp); }
__device__ __forceinline__ float small_rcp(int d) { return __builtin_amdgcn_rcpf((float)d); }

// Whole planes in LDS for the depthwise kernels, forward and backward: quads of four columns, every row with four zeros before it
// (and so, with those of the next row, after it) and K / 2 rows of zeros above and below. A thread's quad of outputs starts at a
// multiple of four columns, so everything it reads is a few aligned 128-bit reads per row - lanes side by side read 16 bytes side
// by side - where single values four columns apart hit every fourth bank. Reads go up to 12 floats beyond the last plane (kPlaneSlack).
constexpr int kPlaneSlack = 16;
__host__ __device__ constexpr int plane_pitch(int W) { return ((W + 3) >> 2) * 4 + 4; }
__host__ __device__ constexpr int plane_floats(int H, int W, int K) { return (H + 2 * (K / 2)) * plane_pitch(W); }
__host__ __device__ constexpr int planes_in_lds(int H, int W, int K) {            // planes of at most 256 quads that a workgroup takes at a time
    const int quads = H * ((W + 3) >> 2), by_quads = quads > 0 && quads <= kBlock ? kBlock / quads : 0, by_floats = (kSmemFloats - kPlaneSlack) / plane_floats(H, W, K);
    return by_quads < by_floats ? by_quads : by_floats;
}
__device__ __forceinline__ void clear_planes(float* xs, int floats, int tid) {   // floats: a multiple of four
    for (int i = 4 * tid; i < floats + kPlaneSlack; i += 4 * kBlock) *reinterpret_cast<float4*>(xs + i) = make_float4(0.f, 0.f, 0.f, 0.f);
}
// four values of row y from column x on (in a row that is no multiple of four columns the last quad starts four before its end)
__device__ __forceinline__ void store_quad(float* plane, int pitch, int K, int y, int x, float4 v) {
    float* dst = plane + (y + K / 2) * pitch + 4 + x;
    if ((x & 3) == 0) {
        *reinterpret_cast<float4*>(dst) = v;
    } else {
        dst[0] = v.x, dst[1] = v.y, dst[2] = v.z, dst[3] = v.w;
    }
}
// What four outputs of a K x K filter with stride S have above them in one row; v[i] is column 4 - K / 2 + i of `src`. Three columns
// and a stride of 1: the quad itself and one value on either side, otherwise whole quads.
template <int K, int S>
__device__ __forceinline__ void load_row(const float* src, float (&v)[3 * S + K]) {
    if constexpr (K == 3 && S == 1) {
        const float4 f = *reinterpret_cast<const float4*>(src + 4);
        v[0] = src[3], v[1] = f.x, v[2] = f.y, v[3] = f.z, v[4] = f.w, v[5] = src[8];
    } else {
        constexpr int FIRST = 4 - K / 2, N = (FIRST + 3 * S + K + 3) / 4;
        float q[4 * N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const float4 f = *reinterpret_cast<const float4*>(src + 4 * i);
            q[4 * i] = f.x, q[4 * i + 1] = f.y, q[4 * i + 2] = f.z, q[4 * i + 3] = f.w;
        }
#pragma unroll
        for (int i = 0; i < 3 * S + K; ++i) v[i] = q[FIRST + i];
    }
}
// the filter of plane p0 + g
template <int KK>
__device__ __forceinline__ void load_filter(const float* w, int p0, int g, int C, float (&f)[KK]) {
    const int c = p0 % C + g;                                   // p0: of the whole workgroup
    const float* wt = w + (c < C ? c : c % C) * KK;
#pragma unroll
    for (int q = 0; q < KK; ++q) f[q] = wt[q];
}

// dwconv for large tensors of small planes (batches of CIFAR-sized maps): a workgroup takes as many whole
// (image, channel) planes as fit 256 quads of input pixels, stages them in LDS with a border of zeros (one 128-bit load per
// thread; the taps then need no bounds) and every thread computes four outputs side by side, stored with one 128-bit store.
// In a row that is no multiple of four the last quad of the input starts four pixels before the end, and the last quad of the
// output is stored value by value. Vector instructions bound it: with single LDS values (bank conflicts in 2 of 3 LDS cycles), the border
// cleared value by value and divisions by the plane's sizes 5 x 5 on 96 images of 44 channels of 32 x 32 took 12.8 us, with quads 9.1
// (3.8 TB/s); 3 x 3 7.1 - 7.6 and 7.3 - 7.5, on 88 channels of 16 x 16 5.2 and 4.7 (by the device's clock, both in turn).
// ------------------------------------------------------------------------------------
template <int K, int S, bool FIN, class Wait>
__device__ __forceinline__ void dwconv_lds_impl(const DwArgs& a, int tile, float* smem, int tid, bool live, Wait& wait) {
    constexpr int SPAN = 3 * S + K;
    const bool fout = wait.far_out();
    const int HW = a.H * a.W, HWo = a.Ho * a.Wo;
    const int pitch = plane_pitch(a.W), plane = plane_floats(a.H, a.W, K);
    const int G = a.planes_per_tile;
    const int p0 = tile * G, np = live ? min(G, a.total / HWo - p0) : 0;
    const int QW = (a.W + 3) >> 2, QWo = (a.Wo + 3) >> 2;
    const int gi = small_div(tid, small_rcp(a.H * QW)), xrem = tid - gi * (a.H * QW), iy = small_div(xrem, small_rcp(QW)), ix = min(4 * (xrem - iy * QW), a.W - 4);
    const int go = small_div(tid, small_rcp(a.Ho * QWo)), orem = tid - go * (a.Ho * QWo), oy = small_div(orem, small_rcp(QWo)), ox = 4 * (orem - oy * QWo);
    const bool xin = gi < np, oin = go < np;
    float w[K * K];
    load_filter(a.w, p0, min(go, max(np - 1, 0)), a.C, w);   // filter taps: not produced by any task
    wait();
    const float4 x4 = xin ? ldg4_any(a.x, a.x + (size_t)(p0 + gi) * HW + iy * a.W + ix, FIN) : make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();                                            // a previous tile of this workgroup has been read to the end
    clear_planes(smem, G * plane, tid);
    __syncthreads();
    if (xin) store_quad(smem + gi * plane, pitch, K, iy, ix, x4);
    __syncthreads();
    if (!oin) return;
    const float* src = smem + go * plane + oy * S * pitch + ox * S;   // row of tap row 0, four columns before the first output's
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int da = 0; da < K; ++da) {
        float v[SPAN];
        load_row<K, S>(src + da * pitch, v);
#pragma unroll
        for (int db = 0; db < K; ++db)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[j] = fmaf(w[da * K + db], v[j * S + db], acc[j]);   // taps in ascending order, as dwconv_tile
    }
    float* out = a.y + (size_t)(p0 + go) * HWo + oy * a.Wo + ox;
    if (ox + 4 <= a.Wo) {
        stg4_any(a.y, out, make_float4(acc[0], acc[1], acc[2], acc[3]), fout);
    } else {
#pragma unroll
        for (int j = 0; j < 3; ++j)
            if (ox + j < a.Wo) stg(a.y, out + j, acc[j], fout);
    }
}
template <bool FIN, class Wait>
__device__ __forceinline__ void dwconv_lds_tile(const DwArgs& a, int tile, float* smem, int tid, bool live, Wait& wait) {
    if (a.K == 3 && a.S == 1) dwconv_lds_impl<3, 1, FIN>(a, tile, smem, tid, live, wait);
    else if (a.K == 3) dwconv_lds_impl<3, 2, FIN>(a, tile, smem, tid, live, wait);
    else if (a.S == 1) dwconv_lds_impl<5, 1, FIN>(a, tile, smem, tid, live, wait);
    else dwconv_lds_impl<5, 2, FIN>(a, tile, smem, tid, live, wait);
}

#include "ng_train_tiles.inc"

// ------------------------------------------------------------------------------------
// kernel table: id -> argument type, tile function, name
// ------------------------------------------------------------------------------------
// FIN: activations are read with device-scope loads (some operand was produced on another
// XCD) - a template argument, because loads sit in the inner loops. Whether the result is stored
// with device-scope stores (some reader sits on another XCD) is a run-time property of the
// `wait` object: a kernel has a handful of stores, and one variant less per kernel halves the code.
template <int KID> struct KernelOf;
#define NG_KERNEL(KID, ARGS, NAME, ...)                                                        \
    template <> struct KernelOf<KID> {                                                         \
        using Args = ARGS;                                                                     \
        static constexpr const char* name = NAME;                                              \
        template <bool FIN, class Wait>                                                        \
        static __device__ __forceinline__ void tile(const ARGS& a, int t, float* smem, int tid, bool live, Wait& wait) { \
            __VA_ARGS__, FIN > (a, t, smem, tid, live, wait);                                  \
        }                                                                                      \
    };
NG_KERNEL(KID_BN, BnArgs, "bn_act", bn_act_tile < PART_L256)
NG_KERNEL(KID_BN_V4, BnArgs, "bn_act_v4", bn_act_tile < PART_L1024)
NG_KERNEL(KID_BN_R64, BnArgs, "bn_act_r64", bn_act_tile < PART_R64)
NG_KERNEL(KID_BN_R16, BnArgs, "bn_act_r16", bn_act_tile < PART_R16)
NG_KERNEL(KID_ADD_R64, AddArgs, "add_n_r64", add_n_tile < PART_R64)
NG_KERNEL(KID_ADD_R16, AddArgs, "add_n_r16", add_n_tile < PART_R16)
NG_KERNEL(KID_ADD, AddArgs, "add_n", add_n_tile < PART_L256)
NG_KERNEL(KID_ADD_V4, AddArgs, "add_n_v4", add_n_tile < PART_L1024)
NG_KERNEL(KID_CONCAT, ConcatArgs, "concat", concat_tile < false)
NG_KERNEL(KID_CONCAT_V4, ConcatArgs, "concat_v4", concat_tile < true)
NG_KERNEL(KID_DW_K3S1, DwArgs, "dwconv_k3s1", dwconv_tile < 3, 1, 1)
NG_KERNEL(KID_DW_K3S2, DwArgs, "dwconv_k3s2", dwconv_tile < 3, 2, 1)
NG_KERNEL(KID_DW_K5S1, DwArgs, "dwconv_k5s1", dwconv_tile < 5, 1, 1)
NG_KERNEL(KID_DW_K5S2, DwArgs, "dwconv_k5s2", dwconv_tile < 5, 2, 1)
NG_KERNEL(KID_DW_K3S1_P4, DwArgs, "dwconv_k3s1_p4", dwconv_tile < 3, 1, 4)
NG_KERNEL(KID_POOL, PoolArgs, "pool3x3", pool3x3_tile < 1, false)
NG_KERNEL(KID_POOL_P4, PoolArgs, "pool3x3_p4", pool3x3_tile < 4, false)
NG_KERNEL(KID_POOL_ROW_S1, PoolArgs, "pool3x3_col4_s1", pool3x3_col_tile < 1)
NG_KERNEL(KID_POOL_ROW_S2, PoolArgs, "pool3x3_col4_s2", pool3x3_col_tile < 2)
NG_KERNEL(KID_POOL_A, PoolAddArgs, "pool3x3_add", pool3x3_tile < 1, true)
NG_KERNEL(KID_POOL_P4A, PoolAddArgs, "pool3x3_p4_add", pool3x3_tile < 4, true)
NG_KERNEL(KID_PW_D4, PwArgs, "conv1x1_mfma_d4", conv1x1_direct_tile < 4)
NG_KERNEL(KID_PW_D8, PwArgs, "conv1x1_mfma_d8", conv1x1_direct_tile < 8)
NG_KERNEL(KID_PW_D16, PwArgs, "conv1x1_mfma_d16", conv1x1_direct_tile < 16)
NG_KERNEL(KID_PW_64, PwArgs, "conv1x1_mfma_64x64", conv1x1_mfma_tile < 64, 64, 16)
NG_KERNEL(KID_PW_V1, PwArgs, "conv1x1_v1", conv1x1_k4_tile < 1, true, false)
NG_KERNEL(KID_PW_V2, PwArgs, "conv1x1_v2", conv1x1_k4_tile < 2, true, false)
NG_KERNEL(KID_PW_V3, PwArgs, "conv1x1_v3", conv1x1_k4_tile < 3, true, false)
NG_KERNEL(KID_PW_V4, PwArgs, "conv1x1_v4", conv1x1_k4_tile < 4, true, false)
NG_KERNEL(KID_PW_S1, PwArgs, "conv1x1_s1", conv1x1_k4_tile < 1, false, false)
NG_KERNEL(KID_PW_S2, PwArgs, "conv1x1_s2", conv1x1_k4_tile < 2, false, false)
NG_KERNEL(KID_PW_S3, PwArgs, "conv1x1_s3", conv1x1_k4_tile < 3, false, false)
NG_KERNEL(KID_PW_S4, PwArgs, "conv1x1_s4", conv1x1_k4_tile < 4, false, false)
NG_KERNEL(KID_C3_T16S1, C3Args, "conv3x3_t16s1", conv3x3_tile < 16, 1)
NG_KERNEL(KID_C3_T16S2, C3Args, "conv3x3_t16s2", conv3x3_tile < 16, 2)
NG_KERNEL(KID_C3_T8S1, C3Args, "conv3x3_t8s1", conv3x3_tile < 8, 1)
NG_KERNEL(KID_C3_T8S2, C3Args, "conv3x3_t8s2", conv3x3_tile < 8, 2)
NG_KERNEL(KID_C3_M1, C3Args, "conv3x3_mfma_1", conv3x3_k4_tile < 1, false)
NG_KERNEL(KID_C3_M2, C3Args, "conv3x3_mfma_2", conv3x3_k4_tile < 2, false)
NG_KERNEL(KID_C3_M3, C3Args, "conv3x3_mfma_3", conv3x3_k4_tile < 3, false)
NG_KERNEL(KID_C3_M4, C3Args, "conv3x3_mfma_4", conv3x3_k4_tile < 4, false)
NG_KERNEL(KID_PW_V1A, PwAddArgs, "conv1x1_v1_add", conv1x1_k4_tile < 1, true, true)
NG_KERNEL(KID_PW_V2A, PwAddArgs, "conv1x1_v2_add", conv1x1_k4_tile < 2, true, true)
NG_KERNEL(KID_PW_V3A, PwAddArgs, "conv1x1_v3_add", conv1x1_k4_tile < 3, true, true)
NG_KERNEL(KID_PW_V4A, PwAddArgs, "conv1x1_v4_add", conv1x1_k4_tile < 4, true, true)
NG_KERNEL(KID_PW_S1A, PwAddArgs, "conv1x1_s1_add", conv1x1_k4_tile < 1, false, true)
NG_KERNEL(KID_PW_S2A, PwAddArgs, "conv1x1_s2_add", conv1x1_k4_tile < 2, false, true)
NG_KERNEL(KID_PW_S3A, PwAddArgs, "conv1x1_s3_add", conv1x1_k4_tile < 3, false, true)
NG_KERNEL(KID_PW_S4A, PwAddArgs, "conv1x1_s4_add", conv1x1_k4_tile < 4, false, true)
NG_KERNEL(KID_C3_M1A, C3AddArgs, "conv3x3_mfma_1_add", conv3x3_k4_tile < 1, true)
NG_KERNEL(KID_C3_M2A, C3AddArgs, "conv3x3_mfma_2_add", conv3x3_k4_tile < 2, true)
NG_KERNEL(KID_C3_M3A, C3AddArgs, "conv3x3_mfma_3_add", conv3x3_k4_tile < 3, true)
NG_KERNEL(KID_C3_M4A, C3AddArgs, "conv3x3_mfma_4_add", conv3x3_k4_tile < 4, true)
NG_KERNEL(KID_C3_L32, C3Args, "conv3x3_lds_32x128", conv3x3_lds_tile < 32, 128, 16)
NG_KERNEL(KID_C3_L64, C3Args, "conv3x3_lds_64x64", conv3x3_lds_tile < 64, 64, 32)
NG_KERNEL(KID_PW_P32, PwArgs, "conv1x1_patch_32x64", conv1x1_patch_tile < 32, 4)
NG_KERNEL(KID_PW_P64, PwArgs, "conv1x1_patch_64x64", conv1x1_patch_tile < 64, 2)
NG_KERNEL(KID_C3_P64, C3Args, "conv3x3_patch_64x64", conv3x3_patch_tile < 64, 1, 2, 2, c3_patch_pixels(KID_C3_P64), c3_patches(KID_C3_P64))
NG_KERNEL(KID_C3_P96, C3Args, "conv3x3_patch_96x64", conv3x3_patch_tile < 96, 1, 2, 2, c3_patch_pixels(KID_C3_P96), c3_patches(KID_C3_P96))
NG_KERNEL(KID_C3_Q32, C3Args, "conv3x3_patch_32x128_wide", conv3x3_patch_tile < 32, 2, 2, 2, c3_patch_pixels(KID_C3_Q32), c3_patches(KID_C3_Q32))
NG_KERNEL(KID_C3_Q64, C3Args, "conv3x3_patch_64x64_wide", conv3x3_patch_tile < 64, 1, 2, 2, c3_patch_pixels(KID_C3_Q64), c3_patches(KID_C3_Q64))
NG_KERNEL(KID_C3_Q128, C3Args, "conv3x3_patch_64x128_wide", conv3x3_patch_tile < 64, 2, 1, 2, c3_patch_pixels(KID_C3_Q128), c3_patches(KID_C3_Q128))
NG_KERNEL(KID_C3_R32, C3Args, "conv3x3_patch_32x128_large", conv3x3_patch_tile < 32, 4, 1, 1, c3_patch_pixels(KID_C3_R32), c3_patches(KID_C3_R32))
NG_KERNEL(KID_C3_R128, C3Args, "conv3x3_patch_64x128_large", conv3x3_patch_tile < 64, 2, 1, 2, c3_patch_pixels(KID_C3_R128), c3_patches(KID_C3_R128))
NG_KERNEL(KID_C3_SK, C3Args, "conv3x3_mfma_split_k", conv3x3_split_k_tile < c3_patch_pixels(KID_C3_SK))
NG_KERNEL(KID_GEMM_PW_FWD, GemmArgs, "gemm_conv1x1_fwd", gemm_tile < GEMM_PW_FWD)
NG_KERNEL(KID_GEMM_PW_DGRAD, GemmArgs, "gemm_conv1x1_dgrad", gemm_tile < GEMM_PW_DGRAD)
NG_KERNEL(KID_GEMM_PW_WGRAD, GemmArgs, "gemm_conv1x1_wgrad", gemm_tile < GEMM_PW_WGRAD)
NG_KERNEL(KID_PW_WGRAD_PX, GemmArgs, "conv1x1_wgrad_px_16", pw_wgrad_px_tile < 1, false)
NG_KERNEL(KID_PW_WGRAD_PX2, GemmArgs, "conv1x1_wgrad_px_32", pw_wgrad_px_tile < 2, false)
NG_KERNEL(KID_C3_WGRAD_PX, GemmArgs, "conv3x3_wgrad_px_16", pw_wgrad_px_tile < 1, true)
NG_KERNEL(KID_C3_WGRAD_PX2, GemmArgs, "conv3x3_wgrad_px_32", pw_wgrad_px_tile < 2, true)
NG_KERNEL(KID_PW_PX_FWD, GemmArgs, "conv1x1_px_fwd", pw_px_tile < GEMM_PW_FWD)
NG_KERNEL(KID_PW_PX_DGRAD, GemmArgs, "conv1x1_px_dgrad", pw_px_tile < GEMM_PW_DGRAD)
NG_KERNEL(KID_GEMM_C3_FWD, GemmArgs, "gemm_conv3x3_fwd", gemm_tile < GEMM_C3_FWD)
NG_KERNEL(KID_GEMM_C3_DGRAD, GemmArgs, "gemm_conv3x3_dgrad", gemm_tile < GEMM_C3_DGRAD)
NG_KERNEL(KID_GEMM_C3_WGRAD, GemmArgs, "gemm_conv3x3_wgrad", gemm_tile < GEMM_C3_WGRAD)
NG_KERNEL(KID_BN_RAW, BnRawArgs, "bn_act_raw", bn_raw_tile < 0)
NG_KERNEL(KID_BN_DGRAD, BnRawArgs, "bn_act_dgrad", bn_raw_tile < 1)
NG_KERNEL(KID_BN_WGRAD, BnRawArgs, "bn_act_wgrad", bn_wgrad_tile < false)
NG_KERNEL(KID_BN_BACKWARD, BnRawArgs, "bn_act_backward", bn_wgrad_tile < true)
NG_KERNEL(KID_RELU_DGRAD, EltGradArgs, "relu_dgrad", elt_grad_tile < 0)
NG_KERNEL(KID_GAP_DGRAD, EltGradArgs, "global_avgpool_dgrad", elt_grad_tile < 1)
NG_KERNEL(KID_SLICE_PAD, EltGradArgs, "slice_pad", elt_grad_tile < 2)
// kernels without further template arguments
#define NG_KERNEL0(KID, ARGS, NAME, FN)                                                        \
    template <> struct KernelOf<KID> {                                                         \
        using Args = ARGS;                                                                     \
        static constexpr const char* name = NAME;                                              \
        template <bool FIN, class Wait>                                                        \
        static __device__ __forceinline__ void tile(const ARGS& a, int t, float* smem, int tid, bool live, Wait& wait) { \
            FN<FIN>(a, t, smem, tid, live, wait);                                              \
        }                                                                                      \
    };
NG_KERNEL0(KID_GAP, GapArgs, "global_avgpool", global_avgpool_tile)
NG_KERNEL0(KID_DW_LDS, DwArgs, "dwconv_lds", dwconv_lds_tile)
NG_KERNEL0(KID_FC_GEMV, FcArgs, "fc_gemv", fc_gemv_tile)
NG_KERNEL0(KID_CHANNEL_SUM, EltGradArgs, "channel_sum", channel_sum_tile)
NG_KERNEL0(KID_DW_DGRAD, DwGradArgs, "dwconv_dgrad", dw_dgrad_tile)
NG_KERNEL0(KID_DW_DGRAD_LDS, DwGradArgs, "dwconv_dgrad_lds", dw_dgrad_lds_tile)
NG_KERNEL0(KID_DW_WGRAD, DwGradArgs, "dwconv_wgrad", dw_wgrad_tile)
NG_KERNEL0(KID_POOL_DGRAD, PoolGradArgs, "pool3x3_dgrad", pool_dgrad_tile)
NG_KERNEL0(KID_POOL_DGRAD_LDS, PoolGradArgs, "pool3x3_dgrad_lds", pool_dgrad_lds_tile)
NG_KERNEL0(KID_SGD, SgdArgs, "sgd_update", sgd_tile)
NG_KERNEL0(KID_SMALL_GEMM, SmallGemmArgs, "small_gemm", small_gemm_tile)
// Two tasks in one launch (they read the same tensor and neither waits for the other): the workgroups of both are dealt
// out alternately while both have tiles left, so that the two - each bound by latency rather than by bandwidth when it runs
// alone - share the compute units from the start.
template <int KA, int KB, bool FIN, class Wait>
__device__ __forceinline__ void pair_tile(const PairArgs<typename KernelOf<KA>::Args, typename KernelOf<KB>::Args>& p, int tile, float* smem,
                                          int tid, bool live, Wait& wait) {
    const int fewer = min(p.na, p.nb);
    const bool first = tile < 2 * fewer ? (tile & 1) == 0 : p.na > p.nb;
    const int t = tile < 2 * fewer ? tile >> 1 : tile - fewer;
    if (first) KernelOf<KA>::template tile<FIN>(p.a, t, smem, tid, live, wait);
    else if constexpr (KA == KID_DW_DGRAD_LDS) dw_wgrad_impl<true, FIN>(p.b, t, smem, tid, live, wait);
    else KernelOf<KB>::template tile<FIN>(p.b, t, smem, tid, live, wait);
}
using PairDwArgs = PairArgs<DwGradArgs, DwGradArgs>;
using PairPwArgs = PairArgs<GemmArgs, GemmArgs>;
// The input gradient (a) and the weight gradient (b) of a 1 x 1 convolution in one launch. Every block of 16 x 16 or 32 x 32
// weights reads a row block of dY and of X, every 16 rows of dX read all of dY: with 44 channels each tensor is read three
// times. The pixels are cut into the splits of the weight gradient, and everything that reads the pixels of one split runs on
// one XCD (pw_backward_share), so that memory is read once and the rest comes from that XCD's L2.
template <int KB, bool FIN, class Wait>
__device__ __forceinline__ void pw_backward_tile(const PairPwArgs& p, int tile, float* smem, int tid, bool live, Wait& wait) {
    const BackwardShare s = pw_backward_share(tile, p.na, p.nb, p.b.splits);
    if (s.which == SHARE_NONE) return;                          // the whole workgroup (launched alone, never by the resident kernel)
    if (s.which == SHARE_INPUT) {
        const int HW = p.a.Ho * p.a.Wo, quads = p.a.N / HW * ((HW + 3) >> 2);
        const int MT = (p.a.M + 15) >> 4, PG = (quads + 15) >> 4, each = p.b.splits >= kXcdSplits ? (PG + p.b.splits - 1) / p.b.splits : PG;
        const int task = s.part * 4 + (tid >> 6), pg = task / MT;
        pw_px_wave<GEMM_PW_DGRAD, FIN>(p.a, s.split * each + pg, task - pg * MT, live && pg < each && s.split * each + pg < PG, tid, wait);
    } else {
        KernelOf<KB>::template tile<FIN>(p.b, s.part * p.b.splits + s.split, smem, tid, live, wait);
    }
}
#define NG_PAIR(KID, ARGS, NAME, KA, KB)                                                       \
    template <> struct KernelOf<KID> {                                                         \
        using Args = ARGS;                                                                     \
        static constexpr const char* name = NAME;                                              \
        template <bool FIN, class Wait>                                                        \
        static __device__ __forceinline__ void tile(const ARGS& a, int t, float* smem, int tid, bool live, Wait& wait) { \
            pair_tile<KA, KB, FIN>(a, t, smem, tid, live, wait);                               \
        }                                                                                      \
    };
NG_PAIR(KID_PAIR_DW, PairDwArgs, "dwconv_dgrad+wgrad", KID_DW_DGRAD, KID_DW_WGRAD)
NG_PAIR(KID_PAIR_DW_LDS, PairDwArgs, "dwconv_dgrad_lds+wgrad", KID_DW_DGRAD_LDS, KID_DW_WGRAD)
#undef NG_PAIR
NG_KERNEL(KID_PAIR_PW16, PairPwArgs, "conv1x1_px_dgrad+wgrad_16", pw_backward_tile < KID_PW_WGRAD_PX)
NG_KERNEL(KID_PAIR_PW32, PairPwArgs, "conv1x1_px_dgrad+wgrad_32", pw_backward_tile < KID_PW_WGRAD_PX2)
#undef NG_KERNEL
NG_KERNEL0(KID_SGD_BATCH, SgdBatchArgs, "sgd_update_batch", sgd_batch_tile)
#undef NG_KERNEL0

// every kernel id that has a tile function
#define NG_FOR_EACH_KID(X)                                                                                              \
    X(KID_BN) X(KID_BN_V4) X(KID_BN_R64) X(KID_BN_R16) X(KID_ADD) X(KID_ADD_V4) X(KID_ADD_R64) X(KID_ADD_R16)           \
    X(KID_CONCAT) X(KID_CONCAT_V4) X(KID_POOL) X(KID_POOL_P4) X(KID_DW_K3S1_P4) X(KID_DW_K3S1) X(KID_DW_K3S2)           \
    X(KID_DW_K5S1) X(KID_DW_K5S2) X(KID_GAP) X(KID_FC_GEMV)                                                             \
    X(KID_PW_D4) X(KID_PW_D8) X(KID_PW_D16) X(KID_PW_64) X(KID_PW_V1) X(KID_PW_V2)                                      \
    X(KID_PW_V3) X(KID_PW_V4) X(KID_PW_S1) X(KID_PW_S2) X(KID_PW_S3) X(KID_PW_S4) X(KID_C3_T16S1)                       \
    X(KID_C3_T16S2) X(KID_C3_T8S1) X(KID_C3_T8S2) X(KID_C3_M1) X(KID_C3_M2)                                             \
    X(KID_C3_M3) X(KID_C3_M4)                                                                                           \
    X(KID_PW_V1A) X(KID_PW_V2A) X(KID_PW_V3A) X(KID_PW_V4A) X(KID_PW_S1A) X(KID_PW_S2A)                                 \
    X(KID_PW_S3A) X(KID_PW_S4A) X(KID_C3_M1A) X(KID_C3_M2A) X(KID_C3_M3A) X(KID_C3_M4A)                                 \
    X(KID_POOL_A) X(KID_POOL_P4A) X(KID_C3_L32) X(KID_C3_L64)                                                          \
    X(KID_C3_P64) X(KID_C3_P96) X(KID_C3_Q32) X(KID_C3_Q64) X(KID_C3_Q128) X(KID_C3_R32) X(KID_C3_R128) X(KID_C3_SK) X(KID_PW_P32) X(KID_PW_P64)                    \
    X(KID_POOL_ROW_S1) X(KID_POOL_ROW_S2) X(KID_DW_LDS)                                                                               \
    X(KID_GEMM_PW_FWD) X(KID_GEMM_PW_DGRAD) X(KID_GEMM_PW_WGRAD) X(KID_GEMM_C3_FWD) X(KID_GEMM_C3_DGRAD)                \
    X(KID_GEMM_C3_WGRAD) X(KID_SMALL_GEMM) X(KID_PW_PX_FWD) X(KID_PW_PX_DGRAD) X(KID_PW_WGRAD_PX) X(KID_PW_WGRAD_PX2) X(KID_C3_WGRAD_PX) X(KID_C3_WGRAD_PX2) X(KID_BN_RAW) X(KID_BN_DGRAD) X(KID_BN_WGRAD) X(KID_RELU_DGRAD) X(KID_DW_DGRAD) X(KID_DW_DGRAD_LDS)                \
    X(KID_DW_WGRAD) X(KID_POOL_DGRAD) X(KID_POOL_DGRAD_LDS) X(KID_GAP_DGRAD) X(KID_CHANNEL_SUM) X(KID_SLICE_PAD) X(KID_SGD) X(KID_SGD_BATCH) X(KID_BN_BACKWARD) X(KID_PAIR_DW) X(KID_PAIR_DW_LDS) X(KID_PAIR_PW16) X(KID_PAIR_PW32)

// A batch-norm epilogue is written into a task's argument block by type (C3Args or PwArgs, whose `ep` fields sit at
// different offsets): the predicates that name the type must agree with the type the kernel takes.
#define NG_CHECK_ARGS(KID)                                                                                              \
    static_assert(!has_bn_epilogue(KID) || (takes_c3_args(KID) ? std::is_base_of<C3Args, KernelOf<KID>::Args>::value    \
                                                               : std::is_base_of<PwArgs, KernelOf<KID>::Args>::value),  \
                  "takes_c3_args / has_bn_epilogue disagree with the kernel's argument type");
NG_FOR_EACH_KID(NG_CHECK_ARGS)
#undef NG_CHECK_ARGS

}  // namespace
}  // namespace ng
