// Few-rows kernel: the fused RMSNorm + router + earliest exit (paper Eq. (2), Sec. 3.3: the routers on a decode step's
// rows) on packed weights, for calls whose rows are so few that the time is latency, not bandwidth.
//
// What bounds it.  An empty kernel takes 2.75 us per launch back to back; on top of that every hand-over between
// workgroups is a dependent round trip to the level where all XCDs agree (0.5-0.8 us: store acknowledged, counter, load,
// atomic).  The split-k forms cut k over workgroups, so they hand over 128 partial sums per row and reach the exit
// decision after four such trips (two launches: after a launch gap of 1.8-3.4 us).  Here a workgroup takes 16 rows x 16
// COLUMNS and the whole of k (its eight waves split k and meet in LDS): it can finish its columns by itself -- 1/rms,
// bias, SiLU, w2 -- and hands over ONE number per row.  The workgroup that completes a row tile's count adds the C * b / 16
// numbers of each row in a fixed order and writes the logits and the exit layer of all checkpoints: three trips, no
// arrival words, and the second part is one wave's work without a barrier.
// Rows come in through LDS, each wave its own k range by coalesced transfers (512 bytes of a row): fetched straight into
// the matrix cores' operand layout a load touches 64 bytes of each of 16 rows, 2 us more at 16 rows of d = 4096.
// Measured (C = 8, d = 4096, packed weights, us per call back to back; before = split-k in one launch up to 16 rows,
// the pair beyond): 8.7 -> 6.4 at T = 1, 8.8 -> 6.9 at 8, 9.6 -> 7.4 at 16, 11.5 -> 8.6 at 48; width 256, T = 8: 12.7 -> 8.8;
// fp32 rows, T = 4: 12.4 -> 9.4; d = 768, T = 4: 10.0 -> 6.3; d = 1600 (no multiple of 128), C = 12, T = 48: 18.4 -> 8.8.  kFull against the latency kernel: 34.6 -> 8.6 at C = 4, T = 32, d = 1608, 12.2 -> 7.5
// at C = 8, T = 4, 13.2 -> 9.9 at C = 1, T = 1, d = 4104 (terms rounded to the nearest instead: 9.0, 8.0 and 11.8).
// Later: the tick without an L2 invalidate 8.5 -> 7.9 at T = 48; waves without a share of the row load nothing instead of zeros, which cost as much as
// data (6.2 -> 5.7 at C = 5, T = 33, d = 1024, 5.5 -> 5.1 at d = 768, T = 4, 7.3 -> 6.8 at C = 6, T = 20, d = 3072); eight or sixteen waves (launch_few_rows); the first arguments
// as scalars, the last ones fetched during the first loads (6.11 -> 6.01 at T = 1, d = 4096, 5.15 -> 4.92 at d = 768, T = 4, 9.4 -> 9.1 at C = 4, T = 16, d = 8192, fp32 9.75 -> 9.44 at T = 8).
// Every storage type, every width, every hidden size whose rows are whole 16-byte chunks.
#pragma once
#include <type_traits>

#include "device_utils.hpp"
#include "prefill_kernel.hpp"

namespace tide {

constexpr int kFewRows = 16, kFewCols = 16;
constexpr int kFewMaxTiles = 64;         // row tiles of a call: one counter each

// 32-k groups per wave and turn.  More (a whole row of d = 4096 in one turn) costs more in registers and code than the
// second turn's round trip: 6.8 / 7.3 us at T = 8 with 8 / 16 groups.
template <int DT> constexpr int few_groups() { return DT == kF32 ? 4 : 8; }
constexpr int kFewChunks = 32;           // 16-byte chunks of a row per wave and turn: 512 bytes
constexpr int kFewRowsPerTransfer = kWave / kFewChunks;
// dynamic LDS: every wave's share of a turn of `rows` rows (rounded up to whole transfers)
constexpr int few_lds_bytes(int waves, int rows) {
    return waves * ((rows + kFewRowsPerTransfer - 1) / kFewRowsPerTransfer * kFewRowsPerTransfer) * kFewChunks * 16;
}

// acc[16x16] += A[16 x 32] * B[32 x 16]: lane l supplies row / column l % 16 and the 8 consecutive k of quarter l / 16.
template <int DT> __device__ __forceinline__ f32x4 mma_k32(u32x4 a, u32x4 b, f32x4 acc);
template <> __device__ __forceinline__ f32x4 mma_k32<kBF16>(u32x4 a, u32x4 b, f32x4 acc) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}
template <> __device__ __forceinline__ f32x4 mma_k32<kF16>(u32x4 a, u32x4 b, f32x4 acc) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), acc, 0, 0, 0);
}

// ceil(T / 16) <= kFewMaxTiles row tiles per checkpoint, b / 16 column blocks (4, 8 or 16);
// p.zpart: [16 * row tiles][C][b / 16] floats; p.counters: kFewMaxTiles words, zero on entry and on exit.
// blockIdx.x -> (checkpoint, row tile, column block), XCD x taking the x-th eighth of that list: a checkpoint's rows and
// weights stay in one or two L2s.
// kFull (fp32 rows): the whole fp32 value of a row times both terms of the weight, as the latency kernel multiplies them, for the calls
// that are its otherwise.  x = hi + mid + lo, each the upper 16 bits of what the one before leaves: exact (24 bits in three times 8), and fewer vector
// instructions, which bound this form, than rounding to the nearest.  The five small products of the six have an accumulator
// of their own and do not lose bits against the large sum.
// What the first loads need comes in scalar arguments (see SplitkTiling); dims = T | C << 16 | log2(b / 16) << 24, T at most 16 kFewMaxTiles.
template <int DT, int kWaves, bool kFull = false>
__global__ __launch_bounds__(kWaves * kWave, 4) void tide_few_rows_kernel(
    const char* hidden, const u32x4* packed, int64_t ckpt_stride_bytes, int64_t row_stride_bytes, int d, uint32_t dims, const float* b1, const float* w2, const PrefillParams p) {
    typedef __attribute__((address_space(3))) char lds_char;
    typedef __attribute__((address_space(1))) const char glb_char;
    constexpr int kE = Storage<DT>::kBytes, kPl = Compute<DT>::kPlanes;
    constexpr int kLd = DT == kF32 ? 2 : 1;                      // 16-byte chunks per 8 elements of a row
    constexpr int kU = few_groups<DT>();
    static_assert(kU * 32 * kE == kFewChunks * 16, "a wave's turn is kFewChunks chunks of a row");
    static_assert(!kFull || DT == kF32, "16-bit rows are exact in one term");
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ __attribute__((aligned(16))) f32x4 part[kWaves][kWave];
    __shared__ float ssq_part[kWaves][kFewRows];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T = dims & 0xffff, C = dims >> 16 & 0xff, shift = dims >> 24, nbk = 1 << shift, b = nbk * kFewCols;
    const int tiles_per_ckpt = (T + kFewRows - 1) / kFewRows;
    const int items = (C * tiles_per_ckpt) << shift;
    const int per_xcd = (items + 7) >> 3;
    const int item = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || item >= items) return;
    const int ct = item >> shift, nb = item & (nbk - 1);
    const int c = tiles_per_ckpt == 1 ? ct : ct / tiles_per_ckpt;
    const int tile = ct - c * tiles_per_ckpt;
    const int row0 = tile * kFewRows;
    const int rows = min(T - row0, kFewRows);                  // rows in use (at least one)

    const int q = lane >> 4, r = lane & 15;
    const int row_bytes = d * kE;
    const int dpad = (d + 127) & ~127;                           // rows of the packed weights
    const int ng = dpad >> 5;                                    // 32-k groups of the packed weights
    // the packed layout (pack_kernel.hpp) in 32-k groups: quarter q of group g is half q % 2 of 16-k group 2 g + q / 2
    const int half = nb >> 3, cb = (nb >> 1) & 3, j0 = (nb & 1) * 16;
    const size_t plane_bytes = (size_t)dpad * 256;
    const int halves = (b + kBottleneck - 1) / kBottleneck;
    const char* wbase = reinterpret_cast<const char*>(packed) + ((size_t)c * halves + half) * kPl * plane_bytes;
    const uint32_t woff = (uint32_t)(((q >> 1) * 4 + cb) * 64 + (q & 1) * 32 + j0 + r) * 16;
    const char* zeros = reinterpret_cast<const char*>(g_zeros);
    const char* rbase = hidden + (int64_t)c * ckpt_stride_bytes + (int64_t)row0 * row_stride_bytes;
    char* mine = smem + wave * (few_lds_bytes(1, rows));                // this wave's share of the rows
    // this lane's columns of the second layer (16 nb + 4 q + 0..3), first so that nothing waits for them later
    const int col = c * b + nb * kFewCols + 4 * q;
    const f32x4 w2v = *reinterpret_cast<const f32x4*>(w2 + col);
    f32x4 b1v = *reinterpret_cast<const f32x4*>((b1 ? b1 : w2) + col);

    f32x4 acc = f32x4{0, 0, 0, 0};
    [[maybe_unused]] f32x4 small = f32x4{0, 0, 0, 0};            // kFull
    float ssq = 0.0f;
    const int turns = (ng + kWaves * kU - 1) / (kWaves * kU);
    const int rl = lane / kFewChunks, slot = lane % kFewChunks;  // transfer: row within it, chunk slot
    const int rr = min(r, rows - 1);                             // rows that do not exist repeat the last one; never stored
    const char* a_lds = mine + rr * (kFewChunks * 16);
    const int ax = (q * kLd) ^ rr;                               // chunk slot = chunk ^ row: conflict-free reads
    for (int i = 0; i < turns; ++i) {
        const int g0 = (i * kWaves + wave) * kU;                 // this wave's groups (uniform)
        if (g0 >= ng) break;                                     // (nothing is left for this wave: no loads of zeros)
        u32x4 w[kU][kPl];
#pragma unroll
        for (int u = 0; u < kU; ++u)
#pragma unroll
            for (int pl = 0; pl < kPl; ++pl) {
                const char* src = g0 + u < ng ? wbase + (size_t)(g0 + u) * 8192 + pl * plane_bytes : zeros;
                w[u][pl] = *reinterpret_cast<const u32x4*>(src + woff);
            }
        const int k0 = g0 * 32 * kE;                             // first byte of this wave's share of a row
        const bool whole = k0 + kFewChunks * 16 <= row_bytes;    // else: chunks beyond the end of the row are zeros
        for (int t = 0; t < rows; t += kFewRowsPerTransfer) {
            const int row = t + rl, off = k0 + ((slot ^ (row & 15)) << 4);
            const char* src = rbase + (int64_t)min(row, rows - 1) * row_stride_bytes + off;
            if (!whole) src = off < row_bytes ? src : zeros;
            __builtin_amdgcn_global_load_lds((glb_char*)src, (lds_char*)(mine + t * kFewChunks * 16), 16, 0, 0);
        }
        TIDE_FETCH_ARGS8(p.zpart, p.counters, p.inv_d, p.eps, p.exit_layer, p.logits, p.fire_mask, p.no_exit);     // for the end, while the loads are under way
        __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));        // vmcnt(0): the transfers have landed (no other wave reads them)
        asm volatile("" ::: "memory");
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            // W1' first, rows second: the accumulators hold the transposed product, a lane owning one row and 4 columns
            if constexpr (DT == kF32) {
                const u32x4 x0 = *reinterpret_cast<const u32x4*>(a_lds + ((ax ^ (8 * u)) << 4));
                const u32x4 x1 = *reinterpret_cast<const u32x4*>(a_lds + ((ax ^ (8 * u) ^ 1) << 4));
                if constexpr (kFull) {
                    u32x4 ah, am, al;                            // pairs of terms: the upper halves of two values
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const uint32_t a = e < 2 ? x0[2 * e] : x1[2 * e - 4], b = e < 2 ? x0[2 * e + 1] : x1[2 * e - 3];
                        const float ra = __uint_as_float(a) - __uint_as_float(a & 0xffff0000u), rb = __uint_as_float(b) - __uint_as_float(b & 0xffff0000u);
                        const float la = ra - __uint_as_float(__float_as_uint(ra) & 0xffff0000u), lb = rb - __uint_as_float(__float_as_uint(rb) & 0xffff0000u);
                        ah[e] = __builtin_amdgcn_perm(b, a, 0x07060302u);
                        am[e] = __builtin_amdgcn_perm(__float_as_uint(rb), __float_as_uint(ra), 0x07060302u);
                        al[e] = __builtin_amdgcn_perm(__float_as_uint(lb), __float_as_uint(la), 0x07060302u);
                    }
                    small = mma_k32<kBF16>(w[u][1], al, small);
                    small = mma_k32<kBF16>(w[u][0], al, small);
                    small = mma_k32<kBF16>(w[u][1], am, small);
                    small = mma_k32<kBF16>(w[u][0], am, small);
                    small = mma_k32<kBF16>(w[u][1], ah, small);
                    acc = mma_k32<kBF16>(w[u][0], ah, acc);
                } else {
                    float x[8];
#pragma unroll
                    for (int e = 0; e < 4; ++e) { x[e] = __uint_as_float(x0[e]); x[4 + e] = __uint_as_float(x1[e]); }
                    __bf16 hi[8], mid[8];
                    split_bf16(x, 8, hi, mid);
                    bf16x8 h8, m8;
#pragma unroll
                    for (int e = 0; e < 8; ++e) { h8[e] = hi[e]; m8[e] = mid[e]; }
                    const u32x4 ah = __builtin_bit_cast(u32x4, h8), am = __builtin_bit_cast(u32x4, m8);
                    acc = mma_k32<kBF16>(w[u][0], am, acc);      // small terms first (mma_k16_split)
                    acc = mma_k32<kBF16>(w[u][1], ah, acc);
                    acc = mma_k32<kBF16>(w[u][0], ah, acc);
                }
                ssq = chunk_sumsq<kF32>(x1, chunk_sumsq<kF32>(x0, ssq));
            } else {
                const u32x4 a = *reinterpret_cast<const u32x4*>(a_lds + ((ax ^ (4 * u)) << 4));
                acc = mma_k32<DT>(w[u][0], a, acc);
                ssq = chunk_sumsq<DT>(a, ssq);
            }
        }
        __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (3 << 14));   // lgkmcnt(0): the reads are back before the next turn's transfers
        asm volatile("" ::: "memory");
    }

    // ---- the waves' shares of k meet in LDS; wave 0 finishes
    if constexpr (kFull) acc += small;
    part[wave][lane] = acc;
    ssq += __shfl_xor(ssq, 16, kWave);
    ssq += __shfl_xor(ssq, 32, kWave);
    if (lane < kFewRows) ssq_part[wave][lane] = ssq;
    __syncthreads();
    if (wave != 0) return;
    const int t = row0 + r;
    const bool live = t < T;
    const int per_row = C << shift;                            // partial logits of a row
    float* ztile = p.zpart + (size_t)row0 * per_row;
    {
        f32x4 s = part[0][lane];
        float ss = ssq_part[0][r];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) { s += part[w][lane]; ss += ssq_part[w][r]; }
        if (!b1) b1v = f32x4{0, 0, 0, 0};
        const float inv = inv_rms_f32(ss, p.inv_d, p.eps);
        float z = 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) z = fmaf(w2v[e], silu_f32(fmaf(inv, s[e], b1v[e])), z);
        z += __shfl_xor(z, 16, kWave);
        z += __shfl_xor(z, 32, kWave);
        if (lane < kFewRows && live) stage_store(ztile + (size_t)r * per_row + (c << shift) + nb, z);
    }
    stage_writes_done();
    // one tick per workgroup; ordering as in last_arrival, by one wave alone.  The counters of neighbouring row tiles are 64
    // bytes apart: atomics on one line take 14 ns each.
    uint32_t* counter = p.counters + ((tile & 3) << 4) + (tile >> 2);
    uint32_t prev = 0;
    if (lane == 0) prev = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    prev = __builtin_amdgcn_readfirstlane(prev);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    if (prev != (uint32_t)per_row - 1) return;

    // ---- last of the row tile: lane (q, r) takes row r's checkpoints q, q + 4, ...
    if (lane == 0) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // zero for the next call
    float* zr = ztile + (size_t)(live ? r : 0) * per_row;
    uint32_t mask = 0;
    int first = 32, layer = p.no_exit;         // earliest eligible checkpoint that fired, and its layer
    auto finish = [&](auto quads_tag) {
        constexpr int kQ = decltype(quads_tag)::value;           // quads of partial logits per row and checkpoint: b / 64
        constexpr int kBatch = kQ == 4 ? 2 : 4;                  // checkpoints whose loads are in flight together
        for (int cb0 = 0; cb0 < C; cb0 += 4 * kBatch) {
            f32x4 v[kBatch][kQ];
            float b2[kBatch], thr[kBatch];
            int lid[kBatch];
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                const int cc = min(cb0 + 4 * k + q, C - 1);
#pragma unroll
                for (int m = 0; m < kQ; ++m) v[k][m] = stage_load4(zr + (cc << shift) + 4 * m);
                b2[k] = p.tab.b2[cc];
                thr[k] = p.tab.thr_logit[cc];
                lid[k] = p.tab.layer_id[cc];
            }
            // the block is left as it was found: zeros, like state words (see the host's part_stays)
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                const int cc = cb0 + 4 * k + q;
                if (live && cc < C) {
#pragma unroll
                    for (int m = 0; m < kQ; ++m) *reinterpret_cast<f32x4*>(zr + (cc << shift) + 4 * m) = f32x4{0, 0, 0, 0};
                }
            }
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                const int cc = cb0 + 4 * k + q;
                float z = 0.0f;
#pragma unroll
                for (int m = 0; m < kQ; ++m) z += (v[k][m][0] + v[k][m][1]) + (v[k][m][2] + v[k][m][3]);
                z += b2[k];
                if (live && cc < C) {
                    const int64_t o = (int64_t)cc * T + t;
                    const bool f = z > thr[k];
                    if (p.logits) p.logits[o] = z;
                    if (p.prob) p.prob[o] = sigmoid_f32(z);
                    if (p.fire) p.fire[o] = f ? 1 : 0;
                    mask |= (f ? 1u : 0u) << cc;
                    if (f && lid[k] >= p.min_layer && cc < first) { first = cc; layer = lid[k]; }
                }
            }
        }
    };
    if (nbk == 8) finish(std::integral_constant<int, 2>{});
    else if (nbk == 4) finish(std::integral_constant<int, 1>{});
    else finish(std::integral_constant<int, 4>{});
    if (!p.exit_layer) return;
#pragma unroll
    for (int x = 16; x <= 32; x *= 2) {                          // the four lanes of a row
        mask |= __shfl_xor(mask, x, kWave);
        const int first2 = __shfl_xor(first, x, kWave), layer2 = __shfl_xor(layer, x, kWave);
        if (first2 < first) { first = first2; layer = layer2; }
    }
    if (live && q == 0) {
        p.exit_layer[t] = layer;
        if (p.fire_mask) p.fire_mask[t] = mask;
    }
}

}  // namespace tide
