// Decode kernel: the same fused RMSNorm + router + earliest exit (paper Eq. (2), Sec. 3.3:
// every decode step evaluates the routers on the new token's checkpoint states) for a
// handful of rows per call, where the cost is reading C routers' weights and latency.
//
// The d-long contraction of each checkpoint is split over slices of k and groups of columns (raw weights: up to
// 512 k values and 32 columns per workgroup; packed: 128 k values and a 128-column half) so that the
// whole chip pulls the weights at once (raw fp32 W1, no packing pass: with so few rows the
// matrix cores have nothing to amortise).  Each workgroup writes its partial sums of its columns and
// partial sum of squares per token (device-scope stores, no fences); the last workgroup of a
// checkpoint (device-scope counter) reduces them in a fixed order and finishes the router; the last checkpoint to
// report a token selects its earliest exit.  One launch, no host round trip, deterministic sums.
#pragma once
#include <type_traits>

#include "device_utils.hpp"

namespace tide {

struct DecodeParams {
    const char* hidden;
    int64_t ckpt_stride_bytes, row_stride_bytes;
    const float* gamma;   // [C][d] or null
    const float* W1;      // [C][d][b] raw weights, or null when `packed` is given
    const u32x4* packed;  // [C][halves][planes][dpad*16 chunks] packed W1' (gamma folded in), or null
    int dpad;             // rows of the packed weights (d rounded up to whole k-tiles)
    const float* b1;      // [C][b] or null
    const float* w2;      // [C][b]
    int C, T, d, S;       // S slices of k; the last one may be partial (any d with 16-byte rows)
    int slice;            // raw weights: k values per slice, a multiple of 128, at most kDecodeRawSlice (packed weights: kDecodeSlice)
    int b, halves;        // bottleneck width (64, 128, 256) and its 128-column halves
    float eps;
    int32_t min_layer, no_exit;
    float* prob; uint8_t* fire; float* logits;   // [C][T], nullable
    int32_t* exit_layer; uint32_t* fire_mask;    // [T], nullable
    uint64_t* arrive;     // [T] arrival words (see report_and_select), zero on entry and on exit
    float* part;          // [C][S][T][halves*128 + 4]: partial pre-activations, then the partial sum of squares
    uint32_t* counter;    // 64 words (decode_counter), zero on entry, zero on exit
    CheckpointTable tab;
};

constexpr int kDecodeThreads = 256;
constexpr int kDecodeSlice = 128;    // k values per workgroup of the packed kernel
constexpr int kDecodeRawSlice = 512; // most k values per workgroup of the raw kernel, ...
constexpr int kDecodeRawCols = 32;   // ... and its columns
constexpr int kDecodeRawMaxSlices = kMaxHidden / kDecodeRawSlice;    // (decode_cut: as few slices as hold the row)
constexpr int kDecodeTB = 8;         // tokens per pass
constexpr int kPartPad = 4;          // the partial sum of squares, padded to 16 bytes

template <int DT> __device__ __forceinline__ void chunk_to_f32(u32x4 c, float* out);
template <> __device__ __forceinline__ void chunk_to_f32<kF32>(u32x4 c, float* out) {
#pragma unroll
    for (int e = 0; e < 4; ++e) out[e] = __uint_as_float(c[e]);
}
template <> __device__ __forceinline__ void chunk_to_f32<kF16>(u32x4 c, float* out) {
    f16x8 h = __builtin_bit_cast(f16x8, c);
#pragma unroll
    for (int e = 0; e < 8; ++e) out[e] = (float)h[e];
}
template <> __device__ __forceinline__ void chunk_to_f32<kBF16>(u32x4 c, float* out) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        out[2 * e] = __uint_as_float(c[e] << 16);
        out[2 * e + 1] = __uint_as_float(c[e] & 0xffff0000u);
    }
}

// The tail of both decode kernels.  Every workgroup of checkpoint c has written its partial
// pre-activations (and, for column half 0, its partial sum of squares) to p.part; the last one to
// arrive reduces them in a fixed order, finishes the router and reports on the arrival words.
// kTB tokens x 32 column quads leave 256 / (32 kTB) threads per pair: each sums a contiguous share of the slices (loads all in
// flight, surplus ones re-read the last slice), the shares meet in LDS in ascending order.
// The checkpoints' counters lie 64 bytes apart as far as the block of 64 words goes: 32 workgroups per checkpoint tick at once,
// and atomics on one line take 14 ns each (all counters in one line: 3.5 us until the last tick at C = 8).
__device__ __forceinline__ uint32_t* decode_counter(const DecodeParams& p, int c) { return p.counter + ((c & 3) << 4) + (c >> 2); }

template <int kHalves, int kTB>
__device__ __forceinline__ void decode_finish(const DecodeParams& p, int c, int workgroups, int* flag, float* lds) {
    constexpr int part_stride = kHalves * kBottleneck + kPartPad;
    constexpr int kG = kDecodeThreads / (32 * kTB);      // threads per (token, quad): 8, 4, 2 or 1
    const int tid = threadIdx.x;
    stage_writes_done();
    if (!last_arrival(decode_counter(p, c), (uint32_t)workgroups, flag)) return;

    const int q = tid & 31, tl = (tid >> 5) % kTB, g = (tid >> 5) / kTB;
    f32x4 b1v[kHalves], w2v[kHalves];
#pragma unroll
    for (int hf = 0; hf < kHalves; ++hf) {
        const int col = hf * kBottleneck + 4 * q;
        b1v[hf] = f32x4{0, 0, 0, 0};
        w2v[hf] = f32x4{0, 0, 0, 0};
        if (col < p.b) {
            if (p.b1) b1v[hf] = *reinterpret_cast<const f32x4*>(p.b1 + c * p.b + col);
            w2v[hf] = *reinterpret_cast<const f32x4*>(p.w2 + c * p.b + col);
        }
    }
    const int s_begin = g * p.S / kG, s_end = (g + 1) * p.S / kG;
    const float* pc = p.part + (size_t)c * p.S * p.T * part_stride;
    const StageBlock pb(pc);                                     // (a checkpoint's partial results are far below 4 GiB)
    f32x4* shares = reinterpret_cast<f32x4*>(lds);               // [kHalves][kG][kTB][32]
    float* ss_shares = lds + kHalves * kG * kTB * 128;           // [kG][kTB]
    for (int t0 = 0; t0 < p.T; t0 += kTB) {
        const int t = t0 + tl;
        const bool valid = t < p.T;
        const int ts = valid ? t : p.T - 1;
        f32x4 a[kHalves];
        float ssum = 0.0f;
#pragma unroll
        for (int hf = 0; hf < kHalves; ++hf) a[hf] = f32x4{0, 0, 0, 0};
        // kBatch partials in flight per thread, from slice s0 on.  kExact: slices beyond the last are not loaded, else the last one is
        // loaded again (branch-free).
        auto add_batch = [&](int s0, auto batch_tag, auto exact_tag) {
            constexpr int kBatch = decltype(batch_tag)::value;
            constexpr bool kExact = decltype(exact_tag)::value;
            f32x4 v[kHalves][kBatch];
#pragma unroll
            for (int hf = 0; hf < kHalves; ++hf)
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    const uint32_t at = ((uint32_t)(kExact ? s0 + u : min(s0 + u, s_end - 1)) * p.T + ts) * part_stride + hf * kBottleneck + 4 * q;
                    if constexpr (kExact) v[hf][u] = f32x4{0, 0, 0, 0};
                    if (!kExact || s0 + u < s_end) v[hf][u] = pb.load4(4 * at);
                }
            // lane q's slice of the batch
            const float sv = stage_load(pc + ((size_t)min(s0 + min(q, kBatch - 1), s_end - 1) * p.T + ts) * part_stride + kHalves * kBottleneck);
#pragma unroll
            for (int hf = 0; hf < kHalves; ++hf)
#pragma unroll
                for (int u = 0; u < kBatch; ++u) a[hf] += s0 + u < s_end ? v[hf][u] : f32x4{0, 0, 0, 0};
            ssum += xor_reduce_sum<5>(q < kBatch && s0 + q < s_end ? sv : 0.0f);     // fixed order: deterministic
        };
        using std::integral_constant;
        if constexpr (kG == 1) {
            // Eight tokens per pass: a thread has all slices of its token.  As few loads as cover them, batch after batch, and none for a token
            // that does not exist: a surplus load is a round trip past every cache too (us, all of 32 slices loaded against this, raw weights: 29.3 / 28.0 at C = 12, T = 25,
            // d = 4296, 9 slices; 12.2 / 11.9 at C = 16, T = 5, 8 slices).  (Width 256: two workgroups per CU, so smaller batches.)
            constexpr int kMost = kHalves == 2 ? 8 : 32;
            for (int s0 = s_begin; valid && s0 < s_end;) {
                const int left = s_end - s0;
                if (kMost == 32 && left > 16) { add_batch(s0, integral_constant<int, kMost>{}, std::true_type{}); s0 += 32; }
                else if (kMost == 32 && left > 8) { add_batch(s0, integral_constant<int, kMost / 2>{}, std::false_type{}); s0 += 16; }
                else if (left > 4) { add_batch(s0, integral_constant<int, 8>{}, std::false_type{}); s0 += 8; }
                else { add_batch(s0, integral_constant<int, 4>{}, std::false_type{}); s0 += 4; }
            }
        } else {
            // fewer tokens (raw weights only): as small a batch as covers the thread's share.  No batch is compiled in that no share needs: with
            // all up to 32 the kernels for 1 / 2 / 4 tokens, widths up to 128, had 196 / 172 / 172 registers, now 128 / 134 / 163 at most (us, C = 32, f16, T = 1:
            // 7.7 -> 7.4 at d = 640; fp32, T = 4, d = 8192: 41 -> 35).
            constexpr int kMostShare = (kDecodeRawMaxSlices + kG - 1) / kG;          // 4, 8 or 16
            auto add_slices = [&](auto batch_tag) {
                for (int s0 = s_begin; s0 < s_end; s0 += decltype(batch_tag)::value) add_batch(s0, batch_tag, std::false_type{});
            };
            const int share = (p.S + kG - 1) / kG;
            if (kMostShare <= 4 || share <= 4) {
                add_slices(integral_constant<int, 4>{});
            } else if constexpr (kMostShare > 4) {
                if (kMostShare <= 8 || kHalves == 2 || share <= 8) add_slices(integral_constant<int, 8>{});
                else if constexpr (kMostShare > 8 && kHalves == 1) add_slices(integral_constant<int, 16>{});
            }
        }
        if constexpr (kG > 1) {
#pragma unroll
            for (int hf = 0; hf < kHalves; ++hf) shares[((hf * kG + g) * kTB + tl) * 32 + q] = a[hf];
            if (q == 0) ss_shares[g * kTB + tl] = ssum;
            __syncthreads();
            ssum = 0.0f;
#pragma unroll
            for (int i = 0; i < kG; ++i) ssum += ss_shares[i * kTB + tl];
#pragma unroll
            for (int hf = 0; hf < kHalves; ++hf) {
                a[hf] = f32x4{0, 0, 0, 0};
#pragma unroll
                for (int i = 0; i < kG; ++i) a[hf] += shares[((hf * kG + i) * kTB + tl) * 32 + q];
            }
        }
#pragma unroll
        for (int hf = 0; hf < kHalves; ++hf)                     // (columns beyond the width: nobody may have written them)
            if (hf * kBottleneck + 4 * q >= p.b) a[hf] = f32x4{0, 0, 0, 0};
        const float r = 1.0f / sqrtf(ssum / (float)p.d + p.eps);
        float term = 0.0f;
#pragma unroll
        for (int hf = 0; hf < kHalves; ++hf)
#pragma unroll
            for (int j = 0; j < 4; ++j) term += w2v[hf][j] * silu_f32(fmaf(r, a[hf][j], b1v[hf][j]));
        term = xor_reduce_sum<5>(term);
        if (valid && q == 0 && g == 0) {
            const float z = p.tab.b2[c] + term;
            const int64_t o = (int64_t)c * p.T + t;
            const bool f = z > p.tab.thr_logit[c];
            if (p.logits) p.logits[o] = z;
            if (p.prob) p.prob[o] = sigmoid_f32(z);
            if (p.fire) p.fire[o] = f ? 1 : 0;
            if (p.exit_layer)
                report_and_select(p.tab, p.C, c, f, p.min_layer, p.no_exit, p.arrive + t, p.exit_layer + t,
                                  p.fire_mask ? p.fire_mask + t : nullptr);
        }
        if constexpr (kG > 1) __syncthreads();           // (kG > 1 means T <= kTB: one pass; kept for any T)
    }
    if (tid == 0) __hip_atomic_store(decode_counter(p, c), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Raw fp32 weights: a workgroup takes 32 columns (128 bytes of a row of W1: whole lines) and up to 512 k values, so that with the same number of workgroups
// as 128 columns x 128 k makes, a checkpoint's last one has a quarter as many partial results to read.
// kHalves = p.halves as a compile-time value (1 or 2): the width-128 kernel carries no code or
// registers for a second column half.  kTB = tokens per pass: 1, 2, 4 or 8, the smallest that holds T (8 beyond).
// What bounds it: 16 MiB of weights on the whole chip (C = 8, d = 4096: 2-3 us), then the hand-over's round trips.  Measured (fp16, C = 8,
// d = 4096, us per call back to back, weights in the caches): 13.7 / 13.7 / 13.8 / 15.1 at T = 1 / 2 / 4 / 8 with eight tokens' arithmetic always, the weights queued before the rows (loads return in
// order, so nothing was staged until the last weight was there), the counters of all checkpoints in one line and one thread per
// (token, quad) in the finish; 10.3 / 11.2 / 12.4 / 14.9 with 128 columns x 128 k per workgroup (the last one of a checkpoint then reads 66 KiB past every cache at
// T = 4, now 17) and partial results read 8 bytes at a time; now 7.3 / 7.7 / 8.2 / 10.0 (of which the gain's loads, see below, and registers, see decode_finish, about 0.6).
// Before this cut / now: d = 8192, C = 6, T = 8 17.2 / 10.9; width 256, T = 4 16.0 / 9.9; width 64, T = 8 13.1 / 9.4; C = 4, T = 2, d = 2048 7.9 / 6.9; fp32, d = 3072, T = 4 10.2 / 8.1.
// (W1 through bounded loads, so that a slice shorter than 512 costs no surplus ones: 1-3 % faster on few workgroups, up to 8 % slower at width 256 on several per CU.)
template <int DT, int kHalves, int kTB>
__global__ __launch_bounds__(kDecodeThreads) void tide_decode_kernel(const DecodeParams p) {
    constexpr int E = Storage<DT>::kElems;
    constexpr int kChunksPerTok = kDecodeRawSlice / E;       // 64 or 128 chunks of a row at most
    constexpr int kLoads = kDecodeRawSlice / 32;             // float4 weight loads per thread
    constexpr int kXLoads = kTB * kChunksPerTok / kDecodeThreads > 0 ? kTB * kChunksPerTok / kDecodeThreads : 1;
    __shared__ __attribute__((aligned(16))) float xs[kTB][kDecodeRawSlice];   // gamma-scaled inputs of this slice
    __shared__ float ss_lds[kTB][kChunksPerTok / kWave];
    __shared__ __attribute__((aligned(16))) float red[4][kTB][kDecodeRawCols];
    __shared__ __attribute__((aligned(16))) float fin[kHalves * kDecodeThreads * 4 + kDecodeThreads / 32];
    __shared__ int flag;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // consecutive workgroup ids land on consecutive XCDs: keep one checkpoint's weights on
    // one XCD (and in its L2 across calls) whenever the counts allow it
    const int groups = p.b / kDecodeRawCols;
    const int nblk = p.C * p.S * groups;
    const int per_xcd = (nblk + 7) >> 3;
    const int work = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || work >= nblk) return;
    const int c = work / (p.S * groups);
    const int rest = work - c * p.S * groups;
    const int s = rest / groups, grp = rest - s * groups;
    const int k0 = s * p.slice, k_end = min(k0 + p.slice, p.d);
    constexpr int part_stride = kHalves * kBottleneck + kPartPad;

    const char* base = p.hidden + (int64_t)c * p.ckpt_stride_bytes;
    // rows first: loads return in order.  Branch-free (a load that does not count goes to a clamped address or beyond the end of its block, and its value is
    // dropped), so that all of them stay in flight together.  Chunks beyond the slice or the row: zeros.
    // (With the gain's loads under a condition -- there may be none -- each of them was waited for by itself, four to a thread, eight at T > 4.
    // us in a graph of calls, f16, C = 8, d = 4096: 7.6 -> 6.9 at T = 1, 8.3 -> 7.9 at 4, 10.2 -> 9.6 at 8; width 256, C = 28, T = 1 25.2 -> 23.5.  A barrier to the
    // scheduler behind the rows' loads only: with one behind the weights' too the last case takes 24.7.)
    const bool gain = p.gamma != nullptr;
    const BoundedBlock g((gain ? p.gamma : p.W1) + (size_t)c * p.d, gain ? (uint32_t)p.d * 4 : 0);
    u32x4 xv[kXLoads];
    f32x4 gv[kXLoads][E / 4];
    auto load_rows = [&](int t0, int nt) {
#pragma unroll
        for (int i = 0; i < kXLoads; ++i) {
            const int qq = tid + i * kDecodeThreads, t = min(qq / kChunksPerTok, nt - 1), k = k0 + qq % kChunksPerTok * E, ks = k < k_end ? k : k0;
            xv[i] = *reinterpret_cast<const u32x4*>(base + (int64_t)(t0 + t) * p.row_stride_bytes + (int64_t)ks * Storage<DT>::kBytes);
#pragma unroll
            for (int e = 0; e < E; e += 4) gv[i][e / 4] = g.load4((uint32_t)(ks + e) * 4);       // (gamma is aligned to a float only)
        }
    };
    load_rows(0, min(kTB, p.T));
    __builtin_amdgcn_sched_barrier(0);

    // ---- this thread's weights: rows k0 + 16*kk + i, columns 4*jq .. 4*jq+3 of this group; a shorter slice leaves the last threads of k without any ----
    const int kk = tid >> 3, jq = tid & 7;
    const float* w = p.W1 + (size_t)c * p.d * p.b + grp * kDecodeRawCols + 4 * jq;
    const int kw = k0 + kLoads * kk;
    f32x4 wreg[kLoads];
#pragma unroll
    for (int i = 0; i < kLoads; ++i) wreg[i] = *reinterpret_cast<const f32x4*>(w + (size_t)min(kw + i, k_end - 1) * p.b);

    // for the end, while the loads are under way (1 % at T = 1, 2 % at 4, 6 % at width 256; with eight tokens 2 % either way)
    if constexpr (kTB < 8) TIDE_FETCH_ARGS8(p.part, p.counter, p.b1, p.w2, p.eps, p.logits, p.exit_layer, p.arrive);

    for (int t0 = 0; t0 < p.T; t0 += kTB) {
        const int nt = min(kTB, p.T - t0);
        if (t0 > 0) load_rows(t0, nt);
        // ---- stage x * gamma for up to kTB tokens; partial sums of squares of raw x ----
#pragma unroll
        for (int i = 0; i < kXLoads; ++i) {
            const int qq = tid + i * kDecodeThreads, t = qq / kChunksPerTok, ch = qq % kChunksPerTok;
            const bool inside = k0 + ch * E < k_end;
            float f[E];
            chunk_to_f32<DT>(inside ? xv[i] : u32x4{0, 0, 0, 0}, f);
            float sq = 0.0f;
#pragma unroll
            for (int e = 0; e < E; ++e) sq = fmaf(f[e], f[e], sq);
            if (t < kTB) {
#pragma unroll
                for (int e = 0; e < E; ++e) xs[t][ch * E + e] = f[e] * (gain && inside ? gv[i][e / 4][e % 4] : 1.0f);
            }
            sq = wave_sum(sq);                                   // a wave's 64 chunks are one token's
            if (lane == 0 && t < kTB) ss_lds[t][ch / kWave] = sq;
        }
        __syncthreads();

        // ---- partial products over this thread's 16 k values ----
        // (in two halves of eight, added at the end: shorter chains of roundings)
        float acc[kTB][4];
#pragma unroll
        for (int t = 0; t < kTB; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[t][j] = 0.0f;
        float first[kTB][4];
#pragma unroll
        for (int i4 = 0; i4 < kLoads / 4; ++i4) {
            if (i4 == kLoads / 8) {
#pragma unroll
                for (int t = 0; t < kTB; ++t)
#pragma unroll
                    for (int j = 0; j < 4; ++j) { first[t][j] = acc[t][j]; acc[t][j] = 0.0f; }
            }
#pragma unroll
            for (int t = 0; t < kTB; ++t) {
                const f32x4 x = *reinterpret_cast<const f32x4*>(&xs[t][kLoads * kk + 4 * i4]);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[t][j] = fmaf(x[i], kw + 4 * i4 + i < k_end ? wreg[4 * i4 + i][j] : 0.0f, acc[t][j]);
                }
            }
        }
        // lanes 8 apart hold the eight k phases of a wave; then the four waves meet in LDS
#pragma unroll
        for (int t = 0; t < kTB; ++t) {
            f32x4 v;
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = add_xor<32>(add_xor<16>(add_xor<8>(first[t][j] + acc[t][j])));
            if (lane < 8) *reinterpret_cast<f32x4*>(&red[wave][t][4 * jq]) = v;
        }
        __syncthreads();
        // thread (tl, q) owns token tl and columns 4q..4q+3 of the group from here on
        {
            const int tl = tid >> 3, q = tid & 7;
            if (tl < nt) {
                float* dst = p.part + (((size_t)c * p.S + s) * p.T + t0 + tl) * part_stride;
                f32x4 v;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    v[j] = (red[0][tl][4 * q + j] + red[1][tl][4 * q + j]) + (red[2][tl][4 * q + j] + red[3][tl][4 * q + j]);
                stage_store4(dst + grp * kDecodeRawCols + 4 * q, v);
                if (q == 0 && grp == 0) {
                    float sum = ss_lds[tl][0];
#pragma unroll
                    for (int i = 1; i < kChunksPerTok / kWave; ++i) sum += ss_lds[tl][i];
                    stage_store(dst + kHalves * kBottleneck, sum);
                }
            }
        }
        __syncthreads();
    }

    decode_finish<kHalves, kTB>(p, c, p.S * groups, &flag, fin);
}

// The same with pre-packed weights (the serving loop's form: gamma already folded in, half the
// bytes of fp32 weights).  A packed chunk holds, for lane = 32h + j of column block nb and 16-k
// group G, the eight values W1'[16G + 8h + e][32 nb + j]; thread (nb = tid / 64, lane) therefore
// owns ONE column and walks the slice's eight groups, so the four waves split the columns, not k:
// no cross-wave reduction, only lanes l and l^32 (the two k halves of a group) meet.
template <int DT, int kHalves>
__global__ __launch_bounds__(kDecodeThreads) void tide_decode_packed_kernel(const DecodeParams p) {
    constexpr int E = Storage<DT>::kElems;
    constexpr int kChunksPerTok = kDecodeSlice / E;
    constexpr int kGroups = kDecodeSlice / 16;               // 16-k groups per slice
    constexpr int kPlanes = Compute<DT>::kPlanes;            // fp32: W1' = hi plane + mid plane
    __shared__ float xs[kDecodeTB][kDecodeSlice];            // raw inputs of this slice (gamma is in the weights)
    __shared__ float ss_lds[kDecodeTB];
    __shared__ __attribute__((aligned(16))) float fin[kHalves * kDecodeThreads * 4 + kDecodeThreads / 32];
    __shared__ int flag;

    const int tid = threadIdx.x, lane = tid & 63, nb = tid >> 6;
    const int nblk = p.C * p.S * kHalves;
    const int per_xcd = (nblk + 7) >> 3;
    const int work = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (work >= nblk) return;
    const int c = work / (p.S * kHalves);
    const int rest = work - c * p.S * kHalves;
    const int s = rest / kHalves, half = rest - s * kHalves;
    const int k0 = s * kDecodeSlice;
    constexpr int part_stride = kHalves * kBottleneck + kPartPad;

    // ---- this thread's weights: 8 groups x 8 consecutive k of one column, as fp32 ----
    const size_t plane_chunks = (size_t)p.dpad * 16;
    const u32x4* pk = p.packed + ((size_t)c * kHalves + half) * kPlanes * plane_chunks + (size_t)(k0 / 16) * 256 + tid;
    float wv[kGroups][8];
#pragma unroll
    for (int G = 0; G < kGroups; ++G) {
        // groups at and beyond the packed rows (a partial last slice) read as zeros, branch-free
        const bool gok = k0 + 16 * G < p.dpad;
        const size_t goff = gok ? (size_t)G * 256 : 0;
        u32x4 hi = pk[goff];
        if (!gok) hi = u32x4{0, 0, 0, 0};
        if constexpr (DT == kF16) {
            const f16x8 h8 = __builtin_bit_cast(f16x8, hi);
#pragma unroll
            for (int e = 0; e < 8; ++e) wv[G][e] = (float)h8[e];
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                wv[G][2 * e] = __uint_as_float(hi[e] << 16);
                wv[G][2 * e + 1] = __uint_as_float(hi[e] & 0xffff0000u);
            }
            if constexpr (DT == kF32) {
                u32x4 mid = pk[plane_chunks + goff];
                if (!gok) mid = u32x4{0, 0, 0, 0};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    wv[G][2 * e] += __uint_as_float(mid[e] << 16);
                    wv[G][2 * e + 1] += __uint_as_float(mid[e] & 0xffff0000u);
                }
            }
        }
    }

    const char* base = p.hidden + (int64_t)c * p.ckpt_stride_bytes + (int64_t)k0 * Storage<DT>::kBytes;
    const int h8 = (lane >> 5) * 8;                          // this lane's k offset within a group
    for (int t0 = 0; t0 < p.T; t0 += kDecodeTB) {
        const int nt = min(kDecodeTB, p.T - t0);
        for (int q = tid; q < kDecodeTB * kChunksPerTok; q += kDecodeThreads) {
            const int t = q / kChunksPerTok, ch = q - t * kChunksPerTok;
            u32x4 v = {0, 0, 0, 0};
            const bool inside = k0 + ch * E < p.d;
            if (t < nt && inside) v = *reinterpret_cast<const u32x4*>(base + (int64_t)(t0 + t) * p.row_stride_bytes + ch * 16);
            float f[E];
            chunk_to_f32<DT>(v, f);
            float sq = 0.0f;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                sq = fmaf(f[e], f[e], sq);
                xs[t][ch * E + e] = f[e];
            }
            sq = xor_reduce_sum<(kChunksPerTok == 16 ? 4 : 5)>(sq);
            if (ch == 0) ss_lds[t] = sq;
        }
        __syncthreads();

        float acc[kDecodeTB];
#pragma unroll
        for (int t = 0; t < kDecodeTB; ++t) acc[t] = 0.0f;
#pragma unroll
        for (int G = 0; G < kGroups; ++G) {
#pragma unroll
            for (int t = 0; t < kDecodeTB; ++t) {
                const f32x4 x0 = *reinterpret_cast<const f32x4*>(&xs[t][16 * G + h8]);
                const f32x4 x1 = *reinterpret_cast<const f32x4*>(&xs[t][16 * G + h8 + 4]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    acc[t] = fmaf(x0[e], wv[G][e], acc[t]);
                    acc[t] = fmaf(x1[e], wv[G][4 + e], acc[t]);
                }
            }
        }
#pragma unroll
        for (int t = 0; t < kDecodeTB; ++t) {
            const float v = acc[t] + __shfl_xor(acc[t], 32, kWave);
            if (lane < 32 && t < nt) {
                float* dst = p.part + (((size_t)c * p.S + s) * p.T + t0 + t) * part_stride;
                stage_store(dst + half * kBottleneck + 32 * nb + lane, v);
            }
        }
        if (tid < nt && half == 0) {
            float* dst = p.part + (((size_t)c * p.S + s) * p.T + t0 + tid) * part_stride;
            stage_store(dst + kHalves * kBottleneck, ss_lds[tid]);
        }
        __syncthreads();
    }
    decode_finish<kHalves, kDecodeTB>(p, c, p.S * kHalves, &flag, fin);
}

}  // namespace tide
