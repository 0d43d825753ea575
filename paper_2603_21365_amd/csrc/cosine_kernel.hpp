// Calibration labels (paper Sec. 3.1 step 2, Eq. (1)): for every token and checkpoint the
// cosine similarity between the checkpoint's hidden state and the last layer's, and the label
// 1[s > tau].  One, two or four waves per token (rows up to 16 KiB), or one or two workgroups, each keep the
// last layer's row in registers and stream their share of the token's C checkpoint rows past it: those are
// read once, the last layer's row once per unit (from L2 after the first), (C+1)*d elements per token from memory.
#pragma once
#include "device_utils.hpp"

namespace tide {

struct CosineParams {
    const char* hidden;
    int64_t ckpt_stride_bytes, row_stride_bytes;
    const char* final_hidden;
    int64_t final_row_stride_bytes;
    int C, T, d;
    int group_bits;    // a token's checkpoints go to 1 << group_bits units, unit g takes checkpoints g, g + (1 << group_bits), ...
    float tau;
    float* sim;        // [C][T] or null
    uint8_t* label;    // [C][T] or null
};

constexpr int kCosineThreads = 256;
constexpr int kCosineMaxChunks = 16;

// dot product and squared norm of one chunk against another, fp32 accumulation
template <int DT> __device__ __forceinline__ void chunk_dot(u32x4 a, u32x4 b, float& dot, float& na);
template <> __device__ __forceinline__ void chunk_dot<kF32>(u32x4 a, u32x4 b, float& dot, float& na) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float x = __uint_as_float(a[e]), y = __uint_as_float(b[e]);
        dot = fmaf(x, y, dot);
        na = fmaf(x, x, na);
    }
}
// 16-bit forms: packed dot-product instructions in one asm statement per chunk, closed by the
// wait states a dot result needs before another kind of vector instruction reads or overwrites
// it (see chunk_sumsq in device_utils.hpp).
#define TIDE_CHUNK_DOT_ASM(op)                                                                        \
    asm(op " %0, %2, %6\n\t" op " %1, %2, %2\n\t" op " %0, %3, %7\n\t" op " %1, %3, %3\n\t"           \
        op " %0, %4, %8\n\t" op " %1, %4, %4\n\t" op " %0, %5, %9\n\t" op " %1, %5, %5\n\ts_nop 3"     \
        : "+v"(dot), "+v"(na)                                                                         \
        : "v"(a.x), "v"(a.y), "v"(a.z), "v"(a.w), "v"(b.x), "v"(b.y), "v"(b.z), "v"(b.w))
template <> __device__ __forceinline__ void chunk_dot<kF16>(u32x4 a, u32x4 b, float& dot, float& na) {
    TIDE_CHUNK_DOT_ASM("v_dot2c_f32_f16");
}
template <> __device__ __forceinline__ void chunk_dot<kBF16>(u32x4 a, u32x4 b, float& dot, float& na) {
    TIDE_CHUNK_DOT_ASM("v_dot2c_f32_bf16");
}
#undef TIDE_CHUNK_DOT_ASM

// kChunks = 16-byte chunks of a row held per thread (the host picks the smallest instantiation that covers the row: three rows'
// worth of registers decide the occupancy, and a surplus chunk is a load all the same).  A token's checkpoints are dealt out to
// 1 << group_bits units (waves of one workgroup, or workgroups of one XCD).
template <int DT, bool kWavePerRow, int kChunks>
__global__ __launch_bounds__(kCosineThreads) void tide_cosine_kernel(
    const char* hidden, int64_t ckpt_stride_bytes, int64_t row_stride_bytes, const char* final_hidden, int64_t final_row_stride_bytes, int T, int d, uint32_t ckpts,
    const CosineParams p) {        // (the first arguments as scalars, see SplitkTiling: 9.8 -> 9.5 us at C = 10, T = 400, d = 5120; ckpts = C | group_bits << 16)
    __shared__ float part[2][4][2];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // scalar: a row's base is, too
    const int C = ckpts & 0xffff, group_bits = ckpts >> 16, step = 1 << group_bits;
    int t, c0;
    if (kWavePerRow) {
        const int unit = blockIdx.x * 4 + wave;
        t = unit >> group_bits;
        c0 = unit & (step - 1);
    } else {
        const int u = blockIdx.x >> 3;                              // workgroup ids 8 apart share an XCD, whose L2 has the last layer's row
        t = ((u >> group_bits) << 3) | (blockIdx.x & 7);
        c0 = u & (step - 1);
    }
    const bool live = t < T;
    const int tt = live ? t : T - 1;             // dead waves shadow the last token and store nothing
    const int nchunk = d * Storage<DT>::kBytes / 16;
    const int stride = kWavePerRow ? kWave : kCosineThreads;
    const int first = kWavePerRow ? lane : tid;

    auto reduce2 = [&](float& a, float& b, int slot) {
        a = wave_sum(a);
        b = wave_sum(b);
        if (!kWavePerRow) {
            if (lane == 0) { part[slot][wave][0] = a; part[slot][wave][1] = b; }
            __syncthreads();
            a = (part[slot][0][0] + part[slot][1][0]) + (part[slot][2][0] + part[slot][3][0]);
            b = (part[slot][0][1] + part[slot][1][1]) + (part[slot][2][1] + part[slot][3][1]);
        }
    };
    // The next checkpoint's row is requested before this one's is reduced, so that a wave
    // always has a row in flight.
    uint32_t at[kChunks];                          // byte offsets of the thread's chunks, clamped: in bounds and branch-free
#pragma unroll
    for (int j = 0; j < kChunks; ++j) at[j] = 16u * (uint32_t)min(first + j * stride, nchunk - 1);
    auto fetch = [&](int c, u32x4 (&x)[kChunks]) {
        const char* row = hidden + (int64_t)c * ckpt_stride_bytes + (int64_t)tt * row_stride_bytes;
#pragma unroll
        for (int j = 0; j < kChunks; ++j) {
            const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(row + at[j]));
            x[j] = first + j * stride < nchunk ? v : u32x4{0, 0, 0, 0};
        }
    };

    const char* fin = final_hidden + (int64_t)tt * final_row_stride_bytes;
    u32x4 y[kChunks], xa[kChunks], xb[kChunks];
    float nl = 0.0f, unused = 0.0f;
#pragma unroll
    for (int j = 0; j < kChunks; ++j) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(fin + at[j]);
        y[j] = first + j * stride < nchunk ? v : u32x4{0, 0, 0, 0};
    }
    fetch(c0, xa);
#pragma unroll
    for (int j = 0; j < kChunks; ++j) nl = chunk_sumsq<DT>(y[j], nl);
    reduce2(nl, unused, 0);

    auto finish = [&](int c, const u32x4 (&x)[kChunks], int slot) {
        float dot = 0.0f, nk = 0.0f;
#pragma unroll
        for (int j = 0; j < kChunks; ++j) chunk_dot<DT>(x[j], y[j], dot, nk);
        reduce2(dot, nk, slot);                    // alternate the LDS slot so one barrier per checkpoint suffices
        const float s = dot / (sqrtf(nk) * sqrtf(nl));
        if (live && (kWavePerRow ? lane == 0 : tid == 0)) {
            const int64_t o = (int64_t)c * T + t;
            if (p.sim) p.sim[o] = s;
            if (p.label) p.label[o] = s > p.tau ? 1 : 0;
        }
    };
    for (int c = c0; c < C; c += 2 * step) {
        if (c + step < C) fetch(c + step, xb);
        finish(c, xa, 1);
        if (c + step < C) {
            if (c + 2 * step < C) fetch(c + 2 * step, xa);
            finish(c + step, xb, 0);
        }
    }
}

}  // namespace tide
