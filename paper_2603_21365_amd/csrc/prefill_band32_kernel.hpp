// Prefill kernel, band form for fp32 rows: the computation of prefill_wide32_kernel.hpp (paper Eq. (2), Sec. 3.4 kernel 1,
// Fig. 1 inference step 3) on tiles of VARIABLE height, as prefill_band_kernel.hpp has it for 16-bit rows.
//
// Why.  The wide-tile kernel wants 256 rows per CU; below that the register-ring kernel took the batch in 64-row tiles, which
// fetch W1' four times as often, write every converted row through LDS twice, and leave the second of two tiles per CU half empty.
// Here a batch of any size is one tile per CU.  With up to four blocks of 32 rows (kMaxBlocks = 4) a block has TWO consumer waves,
// each half of every stage's k: a wave alone on its SIMD hides neither its conversions nor its LDS reads behind its matrix steps,
// and the two waves' accumulators meet once per tile, in LDS.  What bounds it: three matrix steps per value and the W1' every wave
// reads from LDS (64 of the 112 KiB that cross LDS per 16 KiB of rows); 4.2 TB/s at four blocks against 4.5 at eight.
// Measured (us, against the forms it replaces, before its fragments were read a step ahead, see Wide32Steps): d = 2560, C = 10, T = 3001 87 -> 79 (one wave
// per block instead of two: 84); d = 4096, C = 8: 111 -> 94 at T = 2300, 132 -> 122 at 4096.  A ring of rows of six or seven stages (the exchange area in its
// slots) was no faster, with the read-ahead or without (76.0 / 77.4): the memory's latency is covered.
// kRagged as in prefill_band_kernel.hpp.  Bottleneck widths 64 / 128.
#pragma once
#include <type_traits>

#include "device_utils.hpp"
#include "prefill_band_kernel.hpp"
#include "prefill_wide32_kernel.hpp"

namespace tide {

// Schedule: every checkpoint gets grid / C workgroups (a tile costs a wave the same time whatever its height, so a band that
// crossed a checkpoint's end would take two tiles' time), each an equal share (+-1) of the checkpoint's U = ceil(T / 32) blocks,
// cut into as few tiles of at most kMaxBlocks blocks as cover it.  Workgroup `block` is number (block % 8) * grid / 8 + block / 8 of
// the checkpoint-major list, so an XCD's L2 holds one or two W1' at a time.
template <int kMaxBlocks>
struct Band32Walk {
    int c, cur, end;
    __host__ __device__ Band32Walk(int block, int grid, int C, int U) {
        const int L = (block & 7) * (grid >> 3) + (block >> 3), per_ckpt = grid / C, j = L % per_ckpt;
        c = L / per_ckpt;
        cur = c < C ? (int)((int64_t)j * U / per_ckpt) : 0;
        end = c < C ? (int)((int64_t)(j + 1) * U / per_ckpt) : 0;
    }
    __host__ __device__ bool valid() const { return cur < end; }
    __host__ __device__ BandTile current() const {
        const int len = end - cur, n = (len + kMaxBlocks - 1) / kMaxBlocks;
        return BandTile{c, cur, (len + n - 1) / n};
    }
    __host__ __device__ void advance() { cur += current().blocks; }
};

// Blocks per tile at most: 4, with two waves to a block, while every workgroup's share is that much at most, else 8.
inline int band32_max_blocks(int C, int U, int grid) {
    const int per_ckpt = grid / C;
    return (U + per_ckpt - 1) / per_ckpt <= 4 ? 4 : 8;
}

template <int kMaxBlocks> constexpr int band32_stages() { return kMaxBlocks == 4 ? 4 : 3; }
template <int kMaxBlocks> constexpr int band32_lds_bytes() {
    // rings, then per-wave 1/rms (8 blocks) or the exchange area of the two k halves (4 blocks)
    return band32_stages<kMaxBlocks>() * (kMaxBlocks * 32 * kWideTileBytes + kWide32BBytes) + (kMaxBlocks == 4 ? 4 * 8192 : 8 * 32 * (int)sizeof(float));
}

template <bool kRagged, int kMaxBlocks>
__global__ __launch_bounds__(kWideThreads, 1) void tide_prefill_band_f32_kernel(const PrefillParams p) {
    typedef __attribute__((address_space(3))) char lds_char;
    typedef __attribute__((address_space(1))) const char glb_char;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr bool kPair = kMaxBlocks == 4;                      // two waves per block, each half of a stage's k
    constexpr int kStages = band32_stages<kMaxBlocks>(), kABytes = kMaxBlocks * 32 * kWideTileBytes;
    constexpr int kBInstr = kWide32PlaneBytes / 1024;            // transfers per plane of W1' and stage: 8
    char* a_ring = smem;
    char* b_ring = smem + kStages * kABytes;
    float* scratch = reinterpret_cast<float*>(b_ring + kStages * kWide32BBytes);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nstage = p.dpad * 4 / kWideTileBytes;              // k-tiles of a row
    typedef Band32Walk<kMaxBlocks> Walk;
    Walk walk((int)blockIdx.x, (int)gridDim.x, p.C, p.tiles_per_ckpt);
    if (!walk.valid()) return;                                   // (the whole workgroup, before any barrier)
    const unsigned band_index = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    auto first_stage = [&](int nth_tile) { return (int)(((band_index + (unsigned)nth_tile) * 7u) % (unsigned)nstage); };
    const size_t plane_chunks = (size_t)p.dpad * 16;             // 16-byte chunks of one plane of a checkpoint's W1'

    if (wave == kWideConsumers + 2) {
        // ------------------------------------------------------------------ the W1' producer: both planes of a stage
        Walk fetch = walk;
        int f_k = 0, f_rot = 0, f_tile = 0, issued = 0;
        const char* bp = nullptr;
        auto aim = [&](const BandTile& t) {
            bp = reinterpret_cast<const char*>(p.packed + (size_t)t.c * 2 * plane_chunks) + lane * 16;
            f_rot = first_stage(f_tile++);
            f_k = 0;
        };
        aim(fetch.current());
        bool fetch_done = false;
        auto issue_next = [&]() {
            if (fetch_done) return;
            int ks = f_k + f_rot;
            ks = ks >= nstage ? ks - nstage : ks;
            char* dst = b_ring + (issued % kStages) * kWide32BBytes;
#pragma unroll
            for (int pl = 0; pl < 2; ++pl)
#pragma unroll
                for (int i = 0; i < kBInstr; ++i)
                    __builtin_amdgcn_global_load_lds((glb_char*)(bp + (int64_t)pl * plane_chunks * 16 + (int64_t)ks * kWide32PlaneBytes + i * 1024),
                                                     (lds_char*)(dst + pl * kWide32PlaneBytes + i * 1024), 16, 0, 0);
            ++issued;
            if (++f_k == nstage) {
                fetch.advance();
                if (fetch.valid()) aim(fetch.current());
                else fetch_done = true;
            }
        };
        for (int s = 0; s < kStages - 1; ++s) issue_next();
        int handed = 0;
        for (; walk.valid(); walk.advance()) {
            for (int k = 0; k < nstage; ++k) {
                // stage `handed` has landed once at most the younger stages' transfers are outstanding
                if (issued - handed == kStages - 1)
                    __builtin_amdgcn_s_waitcnt(vmcnt_imm((kStages - 2) * 2 * kBInstr));
                else
                    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
                ring_barrier();
                ++handed;
                issue_next();
            }
            if constexpr (kPair) { ring_barrier(); ring_barrier(); ring_barrier(); }   // the consumers' epilogue
        }
        return;
    }
    if (wave >= kWideConsumers) {
        // ------------------------------------------------------------------ row producers (organised as in prefill_band_kernel.hpp)
        const int pw = wave - kWideConsumers;
        const int rl = lane / kWideChunksPerRow, slot = lane % kWideChunksPerRow;
        const int whole_stages = p.d * 4 / kWideTileBytes;       // kRagged: stages from here on reach beyond the end of the rows
        int issued = 0, handed = 0, in_tile = 0, f_tile = 0;
        // transfers of the stages in flight behind the one handed over next: counts per stage, youngest last
        int cnt[kStages - 1];
#pragma unroll
        for (int i = 0; i < kStages - 1; ++i) cnt[i] = 0;
        auto end_of_consumed_tile = [&]() {
            ++handed;
            if constexpr (kPair) {
                if (++in_tile == nstage) {
                    in_tile = 0;
                    ring_barrier();                    // the three barriers of the consumers' epilogue
                    ring_barrier();
                    ring_barrier();
                }
            }
        };
        auto younger = [&]() { int n = 0; for (int i = 1; i < kStages - 1; ++i) n += cnt[i]; return n; };   // than the oldest in flight
        auto push = [&](int n) {
#pragma unroll
            for (int i = 0; i + 1 < kStages - 1; ++i) cnt[i] = cnt[i + 1];
            cnt[kStages - 2] = n;
        };
        auto fetch_tile = [&](auto blocks_tag, const BandTile& t) {
            constexpr int kN = decltype(blocks_tag)::value;
            const char* base = p.hidden + (int64_t)t.c * p.ckpt_stride_bytes;
            const int row0 = t.block0 * 32;
            const char* gp[2 * kN];
            int cx[2 * kN];                                      // byte of the row segment this lane fetches
#pragma unroll
            for (int i = 0; i < 2 * kN; ++i) {
                const int row = (2 * i + pw) * kWideRowsPerTransfer + rl;       // row within the tile
                int r = row0 + row;
                r = r < p.T ? r : p.T - 1;                                      // ragged tail: re-read the last row
                cx[i] = (slot ^ wide_swizzle(row)) << 4;
                gp[i] = base + (int64_t)r * p.row_stride_bytes + cx[i];
            }
            const int rot = first_stage(f_tile++);
            for (int k = 0; k < nstage; ++k) {
                const bool hand = issued >= kStages - 1;                       // (false for the first stages of the band only)
                if (hand) {
                    if (k < kStages - 2) band_wait_vmcnt(younger());            // stages of the tile before among those in flight
                    else __builtin_amdgcn_s_waitcnt(vmcnt_imm((kStages - 2) * 2 * kN));
                    ring_barrier();
                }
                int ks = k + rot;
                ks = ks >= nstage ? ks - nstage : ks;
                char* dst = a_ring + (issued % kStages) * kABytes + pw * 1024;
                const int64_t koff = (int64_t)ks * kWideTileBytes;
                if (kRagged && ks >= whole_stages) {
                    const char* zeros = reinterpret_cast<const char*>(g_zeros);
#pragma unroll
                    for (int i = 0; i < 2 * kN; ++i)
                        __builtin_amdgcn_global_load_lds((glb_char*)((int)koff + cx[i] < p.d * 4 ? gp[i] + koff : zeros), (lds_char*)(dst + i * 2048), 16, 0, 0);
                } else {
                    row_transfers<kRagged>(p.shared_lines, [&](auto policy) {
#pragma unroll
                        for (int i = 0; i < 2 * kN; ++i)
                            __builtin_amdgcn_global_load_lds((glb_char*)(gp[i] + koff), (lds_char*)(dst + i * 2048), 16, 0, decltype(policy)::value);
                    });
                }
                ++issued;
                push(2 * kN);
                if (hand) end_of_consumed_tile();
            }
        };
        for (Walk fetch = walk; fetch.valid(); fetch.advance()) {
            const BandTile t = fetch.current();
            switch (t.blocks) {
            case 8: if constexpr (kMaxBlocks >= 8) fetch_tile(std::integral_constant<int, 8>{}, t); break;
            case 7: if constexpr (kMaxBlocks >= 8) fetch_tile(std::integral_constant<int, 7>{}, t); break;
            case 6: if constexpr (kMaxBlocks >= 8) fetch_tile(std::integral_constant<int, 6>{}, t); break;
            case 5: if constexpr (kMaxBlocks >= 8) fetch_tile(std::integral_constant<int, 5>{}, t); break;
            case 4: fetch_tile(std::integral_constant<int, 4>{}, t); break;
            case 3: fetch_tile(std::integral_constant<int, 3>{}, t); break;
            case 2: fetch_tile(std::integral_constant<int, 2>{}, t); break;
            default: fetch_tile(std::integral_constant<int, 1>{}, t); break;
            }
        }
        // the stages still in flight (a row has at least kStages of them: d >= 128)
        while (handed < issued) {
            band_wait_vmcnt(younger());
            ring_barrier();
            push(0);
            end_of_consumed_tile();
        }
        return;
    }

    // ---------------------------------------------------------------------- consumers: wave w owns block w of the tile (kPair: block w % 4,
    // the 16-k group w / 4 of every stage)
    const int r = lane & 31, h = lane >> 5;
    const int wb = kPair ? wave & 3 : wave, kg = kPair ? wave >> 2 : 0;
    const int a_row = (32 * wb + r) * kWideTileBytes;
    const int a_swz = wide_swizzle(r);
    float* my_rms = scratch + wave * 32;                         // (not kPair)
    const int vsel = (lane >> 1) & 15;
    const int my_row = 8 * (vsel >> 2) + 4 * h + (vsel & 3);    // the row whose total reduce_scatter16 leaves in this lane
    const int wave_u = __builtin_amdgcn_readfirstlane(wb), kg_u = __builtin_amdgcn_readfirstlane(kg);
    int stage = 0;
    for (; walk.valid(); walk.advance()) {
        const BandTile t = walk.current();
        if (wave_u >= t.blocks) {                                // no block for this wave: it keeps the barriers
            for (int k = 0; k < nstage + (kPair ? 3 : 0); ++k) ring_barrier();
            stage += nstage;
            continue;
        }
        const int c = t.c, row0 = (t.block0 + wb) * 32;
        Wide32Steps steps;
        steps.clear();
        auto read = [&](int g, auto multiply_tag) {
            steps.template advance<decltype(multiply_tag)::value>(a_ring + (stage % kStages) * kABytes + a_row, b_ring + (stage % kStages) * kWide32BBytes + lane * 16, g, h, a_swz);
        };
        ring_barrier();
        read(kPair ? kg_u : 0, std::false_type{});
        if constexpr (!kPair) read(1, std::true_type{});
        ++stage;
        for (int k = 1; k < nstage; ++k) {
            wide32_hand_over();
            read(kPair ? kg_u : 0, std::true_type{});
            if constexpr (!kPair) read(1, std::true_type{});
            ++stage;
        }
        steps.finish();
        f32x16 (&acc)[4] = steps.acc;
        const float ssq = steps.ssq;
        float xs[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) xs[v] = 0.0f;
        const float s2 = ssq + __shfl_xor(ssq, 32, kWave);       // lanes l and l^32 hold the two halves of row l % 32
        // columns of block nb of this wave's rows, 1/rms of a quad's four rows at rs4(q); columns at and beyond the bottleneck width
        // are zero padding: their w2 is zero
        auto columns = [&](const f32x16& a16, int nb, auto rs4) {
            const int col = 32 * nb + r;
            const float b1c = (p.b1 && col < p.b) ? p.b1[c * p.b + col] : 0.0f;
            const float w2c = col < p.b ? p.w2[c * p.b + col] : 0.0f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {                  // registers 4q..4q+3 are rows 8q + 4h + (0..3) of the block
                const f32x4 rs = rs4(q);
#pragma unroll
                for (int e = 0; e < 4; ++e) xs[4 * q + e] += w2c * silu_f32(fmaf(rs[e], a16[4 * q + e], b1c));
            }
        };
        if constexpr (!kPair) {
            // ---- epilogue, all within the wave
            if (lane < 32) my_rms[lane] = inv_rms_f32(s2, p.inv_d, p.eps);
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) columns(acc[nb], nb, [&](int q) { return *reinterpret_cast<const f32x4*>(my_rms + 8 * q + 4 * h); });
            const float total = reduce_scatter16(xs, lane);    // the sum over this wave's 32 lanes = all 128 columns
            if (!(lane & 1)) {
                const int tok = row0 + my_row;
                if (tok < p.T) emit_router_result(p, c, tok, p.tab.b2[c] + total);
            }
        } else {
            // ---- epilogue of two waves: the first half of k finishes column blocks 0 and 1, the second half 2 and 3.  The pair's
            // 8 KiB of the exchange area carry 0 and 1 one way, then 2 and 3 the other.
            float* ex = scratch + wb * 2048 + lane * 4;
            auto put = [&](int nb0) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        *reinterpret_cast<f32x4*>(ex + (i * 4 + q) * 256) = f32x4{acc[nb0 + i][4 * q], acc[nb0 + i][4 * q + 1], acc[nb0 + i][4 * q + 2], acc[nb0 + i][4 * q + 3]};
            };
            auto add = [&](int nb0) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const f32x4 v = *reinterpret_cast<const f32x4*>(ex + (i * 4 + q) * 256);
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[nb0 + i][4 * q + e] += v[e];
                    }
            };
            // sums of squares and logit halves of the pair: in the W1' slot of the stage just consumed, which is refilled only
            // after the next tile's first hand-over
            float* ssx = reinterpret_cast<float*>(b_ring + ((stage - 1) % kStages) * kWide32BBytes) + wb * 96;   // [2][32]
            float* zx = ssx + 64;                                                                                // [32]
            if (kg_u) put(0);
            __syncthreads();
            if (lane < 32) ssx[kg_u * 32 + lane] = s2;
            if (!kg_u) {
                add(0);
                put(2);
            }
            __syncthreads();
            if (kg_u) add(2);
            auto rs4 = [&](int q) {
                const f32x4 s0 = *reinterpret_cast<const f32x4*>(ssx + 8 * q + 4 * h), s1 = *reinterpret_cast<const f32x4*>(ssx + 32 + 8 * q + 4 * h);
                f32x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = inv_rms_f32(s0[e] + s1[e], p.inv_d, p.eps);
                return v;
            };
            if (kg_u) {
                columns(acc[2], 2, rs4);
                columns(acc[3], 3, rs4);
            } else {
                columns(acc[0], 0, rs4);
                columns(acc[1], 1, rs4);
            }
            const float total = reduce_scatter16(xs, lane);
            if (kg_u && !(lane & 1)) zx[my_row] = total;
            __syncthreads();
            if (!kg_u && !(lane & 1)) {
                const int tok = row0 + my_row;
                if (tok < p.T) emit_router_result(p, c, tok, p.tab.b2[c] + (total + zx[my_row]));
            }
        }
    }
}

}  // namespace tide
