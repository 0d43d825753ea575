// Prefill kernel, one-tile form: the full-tile path of prefill_dma_kernel.hpp (paper Eq. (2),
// Sec. 3.4 kernel 1, Fig. 1 inference step 3) and nothing else -- one tile of 128 or 64 rows per
// workgroup, no persistent schedule, no pieces.
//
// Why another form.  When a batch gives every CU one whole tile or none (between half as many
// tiles as CUs and as many), the streaming kernel's schedule has nothing to decide, but its
// code for walking tile lists and for 64- and 32-row pieces still costs registers (241 and 19 spilled scalars against
// 181 here; the forms in bursts, below, spend 237-242 on a second set of W1') and set-up time: this form is 1-3 % faster on such batches (measured at d = 2048,
// 4096 and 8192 on the same box; the 8B-shaped prefill of 8 x 4096 rows is one).  There, keeping W1' two
// k-tiles ahead instead of one, or filling all four ring slots at the start, changes nothing.
// 16-bit storage types, d a multiple of 128 (kRagged: any rows of whole 16-byte chunks, zeros fetched beyond their end).
#pragma once
#include <type_traits>

#include "device_utils.hpp"
#include "prefill_dma_kernel.hpp"

namespace tide {

// Timeline builds (-DTIDE_TILE_TIMELINE; see timeline.py): thread 0 of every workgroup -- lane 0 of consumer
// wave 0 -- notes the 100 MHz real-time counter at its start, at every ring hand-over, at the end of its k
// loop, after the first epilogue barrier, after its share of the epilogue, after the last barrier and once
// its results are acknowledged: kTimelineStamps 64-bit values per workgroup in the buffer tide_debug_timeline set.
#ifdef TIDE_TILE_TIMELINE
constexpr int kTimelineStamps = 48;
__device__ unsigned long long* g_tile_timeline = nullptr;
#define TIDE_STAMP()                                                                              \
    do {                                                                                          \
        if (tid == 0 && tl_base && tl_n < kTimelineStamps) tl_base[tl_n] = __builtin_amdgcn_s_memrealtime(); \
        ++tl_n;                                                                                   \
    } while (0)
#else
#define TIDE_STAMP() do { } while (0)
#endif

constexpr int kTileRows = 128;
// kHalves = 128-column halves of the bottleneck (2 at width 256): 4 consumer waves per half, wave w owning columns
// 32 (w % 4) .. + 31 of half w / 4.  Every wave has columns of its own, so its W1' fragments still come straight from
// L2, once per workgroup; the ring holds rows only.
constexpr int tile_consumers(int kHalves) { return kDmaConsumers * kHalves; }
constexpr int tile_threads(int kHalves) { return (tile_consumers(kHalves) + kDmaProducers) * kWave; }          // 384 / 640
// What bounds the form while HBM does not: a CU has about 32 KiB of loads outstanding, answered in order, whatever they are.  So its rate from memory is 32 KiB per
// latency (measured: 62 GB/s per CU from memory alone, 55 with L2's mixed in finely, where L2 alone gives 180, a limit of its own), and W1' from L2 pays
// the rows' memory latency whenever both are requested in turns.  kBurst: a stage's W1' fragments are requested all at once at its start (two sets of
// registers), the rows in a burst of their own, and no more of them ahead than two stages (four stages instead of three: 2-4 % slower).  Tiles of 64 rows, which read
// twice as much W1' as rows, take two k-tiles per stage, and their producers let W1' go first (some 640 cycles).  us, without / with, bf16, C = 8, rows from memory:
//   64 rows (the streaming kernel before): d = 4096 29.7 / 27.1 at T = 1203, 38.4 / 33.9 at 2040, d = 5120 35.8 / 33.5 at 1250, d = 8192 53.1 / 47.2, d = 1024 12.3 / 11.6 at
//   1500 (one k-tile per stage: 29.1, 37.1 at d = 4096; without the 640 cycles / with: 34.4 / 33.6 at d = 4096, T = 2040, 21.5 / 21.3 at d = 2176, 0.5 % on short rows); an odd number of k-tiles: d = 640 9.45 / 9.15 at 1500, 1600 17.5 / 16.3 at 2040, d = 384 level (its last stage
//   asks for the W1' of its one k-tile twice; a branch round the second half of a stage's requests: 6 % faster there, up to 5 % slower from d = 1920 on);
//   128 rows: d = 4096 43.5 / 41.0 at T = 2100, 47.4 / 45.7 at 3000, but 50.9 / 51.1 at 3500, 55.4 / 56.4 at 4096; d = 2048 24.8 / 23.7, 27.0 / 26.4, 28.4 / 28.7, 30.4 / 32.6; d = 8192
//   79.6 / 75.4, 86.8 / 86.3, 93.2 / 95.5, 102.8 / 107.4 (d = 5120 60.5 / 57.7 at 3000, 68.6 / 68.3 at 4096): with most of the CUs at work HBM bounds it, and
//   the finer mixture keeps that busier -- hence bursts up to three quarters of the CUs (launch_tile).
// (Width 256 has no registers for a second set.)
constexpr int tile_stages(bool burst) { return burst ? 3 : kDmaStages; }
constexpr int tile_k_tiles(int rows) { return rows == 64 ? 2 : 1; }          // per stage
constexpr int tile_lds_bytes(int kHalves, int rows, bool burst) {
    // ring + per-wave row sums of squares (the waves of half 0) + per-wave logit partials
    return tile_stages(burst) * tile_k_tiles(rows) * rows * kTileBytes + (kDmaConsumers + tile_consumers(kHalves)) * rows * (int)sizeof(float);
}

// blockIdx.x -> tile as in the other forms: XCD x (workgroup id mod 8) takes the x-th eighth of the
// checkpoint-major tile list from p.tile_begin on, so that an XCD's L2 holds one W1' at a time.
template <int DT, int kHalves, bool kRagged, int kRowsM, bool kBurst>
__global__ __launch_bounds__(tile_threads(kHalves), 1) void tide_prefill_tile_kernel(const PrefillParams p) {
    static_assert(DT != kF32, "16-bit storage types only");
    static_assert(kRowsM == 128 || (kRowsM == 64 && kBurst), "64 rows: in bursts only");
    static_assert(!kBurst || kHalves == 1, "two sets of W1' fragments");
    typedef __attribute__((address_space(3))) char lds_char;
    typedef __attribute__((address_space(1))) const char glb_char;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr int kBlocks = kRowsM / 32;
    constexpr int kStages = tile_stages(kBurst), kT = tile_k_tiles(kRowsM);       // stages of the ring, k-tiles of a stage
    constexpr int kTileOfRows = kRowsM * kTileBytes, kStageBytes = kT * kTileOfRows;
    constexpr int kInstrPerProducer = kRowsM / 4 / kDmaProducers;   // one transfer = 4 rows x 256 B
    char* ring = smem;
    constexpr int kConsumers = tile_consumers(kHalves);
    float* ss_part = reinterpret_cast<float*>(smem + kStages * kStageBytes);      // [4][kRowsM]
    float* z_part = ss_part + kDmaConsumers * kRowsM;                              // [kConsumers][kRowsM]

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#ifdef TIDE_TILE_TIMELINE
    unsigned long long* tl_base = g_tile_timeline ? g_tile_timeline + (size_t)blockIdx.x * kTimelineStamps : nullptr;
    int tl_n = 0;
#endif
    TIDE_STAMP();
    const int per_xcd = (p.total_tiles - p.tile_begin + 7) >> 3;
    const int tile = p.tile_begin + (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || tile >= p.total_tiles) return;
    const int ntile = p.dpad * Storage<DT>::kBytes / kTileBytes, nstage = (ntile + kT - 1) / kT;
    // Rows are a power-of-two number of bytes apart and all workgroups start together: each tile
    // starts its k loop at a different k-tile and wraps (see prefill_kernel.hpp).
    const int rot = (int)(((unsigned)tile * 5u) % (unsigned)ntile);
    auto kt_of = [&](int k) { const int x = k + rot; return x >= ntile ? x - ntile : x; };
    const int c = tile / p.tiles_per_ckpt;
    const int row0 = (tile - c * p.tiles_per_ckpt) * kRowsM;

    if (wave >= kConsumers) {
        // ------------------------------------------------------------------ producers
        const int pw = wave - kConsumers;
        const int rl = lane >> 4, slot = lane & 15;
        const char* base = p.hidden + (int64_t)c * p.ckpt_stride_bytes;
        const char* gp[kInstrPerProducer];
        const int row_bytes = p.d * Storage<DT>::kBytes, whole = row_bytes / kTileBytes;   // kRagged: k-tiles from `whole` on reach beyond the rows' end
#pragma unroll
        for (int i = 0; i < kInstrPerProducer; ++i) {
            const int row = (pw * kInstrPerProducer + i) * 4 + rl;          // row within the tile
            int r = row0 + row;
            r = r < p.T ? r : p.T - 1;                                      // ragged tail: re-read the last row
            gp[i] = base + (int64_t)r * p.row_stride_bytes + ((slot ^ (row & 15)) << 4);
        }
        int issued = 0;
        auto issue_next = [&]() {
            if (issued >= nstage) return;
#pragma unroll
            for (int h = 0; h < kT; ++h) {
                if (h > 0 && issued * kT + h >= ntile) break;               // (an odd number of k-tiles: the last stage has one)
                char* dst = ring + (issued % kStages) * kStageBytes + h * kTileOfRows;
                const int kt = kt_of(issued * kT + h);
                if (kRagged && kt >= whole) {
#pragma unroll
                    for (int i = 0; i < kInstrPerProducer; ++i) {
                        const int row = (pw * kInstrPerProducer + i) * 4 + rl;
                        const bool inside = kt * kTileBytes + ((slot ^ (row & 15)) << 4) < row_bytes;
                        __builtin_amdgcn_global_load_lds((glb_char*)(inside ? gp[i] + (int64_t)kt * kTileBytes : reinterpret_cast<const char*>(g_zeros)),
                                                         (lds_char*)(dst + (pw * kInstrPerProducer + i) * 1024), 16, 0, 0);
                    }
                } else {
                    row_transfers<kRagged>(p.shared_lines, [&](auto policy) {
#pragma unroll
                        for (int i = 0; i < kInstrPerProducer; ++i)
                            __builtin_amdgcn_global_load_lds((glb_char*)(gp[i] + (int64_t)kt * kTileBytes),
                                                             (lds_char*)(dst + (pw * kInstrPerProducer + i) * 1024), 16, 0, decltype(policy)::value);
                    });
                }
            }
            ++issued;
        };
        constexpr int kPerStage = kT * kInstrPerProducer;                   // transfers
        for (int s = 0; s < kStages - 1; ++s) issue_next();
        for (int k = 0; k < nstage; ++k) {
            // stage k has landed once only the transfers of the younger stages are outstanding (loads complete in issue order)
            const int younger = issued - k - 1;
            static_assert(kT == 1 || kStages == 3, "at most one stage of two k-tiles is younger");
            if (kT == 1 && younger >= 2) __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * kPerStage));
            else if (kT > 1 && younger == 1 && (k + 2) * kT > ntile) __builtin_amdgcn_s_waitcnt(vmcnt_imm(kInstrPerProducer));      // (the last stage, with one k-tile)
            else if (younger == 1) __builtin_amdgcn_s_waitcnt(vmcnt_imm(kPerStage));
            else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
            ring_barrier();                        // stage k handed over; the slot of stage k-1 is free
            if (kRowsM == 64 && issued < nstage) __builtin_amdgcn_s_sleep(10);      // (the consumers' W1' first)
            issue_next();
        }
        ring_barrier();                            // the two barriers of the consumers' epilogue
        ring_barrier();
        return;
    }

    // ---------------------------------------------------------------------- consumers
    const int half = wave >> 2, cw = wave & 3;                   // column half, column block within it
    const int wave_u = __builtin_amdgcn_readfirstlane(cw);       // uniform: branches on it are scalar
    const int half_u = __builtin_amdgcn_readfirstlane(half);
    const int r = lane & 31;
    const int a_base = r * kTileBytes;
    const int y16 = ((lane >> 5) ^ (r & 15)) << 4;               // see prefill_dma_kernel.hpp
    const size_t ckpt_chunks = (size_t)p.dpad * kBottleneck / Storage<DT>::kElems;
    const u32x4* bptr = p.packed + ((size_t)c * kHalves + half) * ckpt_chunks + cw * 64 + lane;
    // The matrix steps take W1' first and the rows second: the accumulators hold the transposed product,
    // a lane owning one row per block and 16 of the wave's 32 columns (router_epilogue_row).  The b1 / w2
    // of those columns are fetched now so that the epilogue does not wait for them (columns at and
    // beyond the bottleneck width are zero padding: their w2 is zero).
    // (With eight consumer waves there are 168 registers per wave and the k loop needs them: there the 32 registers
    // of these constants are fetched after the loop, and the first epilogue barrier covers most of the round trip.)
    auto fetch_ecols = [&]() { return load_epilogue_columns(p.b1 ? p.b1 + c * p.b : nullptr, p.w2 + c * p.b, p.b, kBottleneck * half + 32 * cw, lane); };
    EpilogueColumns ecols;
    if constexpr (kHalves == 1) ecols = fetch_ecols();
    constexpr int kGroups = Compute<DT>::kMmaGroups, kSet = kT * kGroups;         // 16-k groups of a k-tile (8) and of a stage
    u32x4 breg[kBurst ? 2 : 1][kSet];                            // W1' fragments, one stage ahead
    // Fragment g of stage s; without bursts s is the k-tile itself, worked out once for its eight fragments (width 256, T = 4096: 80.1 / 78.6 us).
    auto fragment = [&](int s, int g) {
        if constexpr (kBurst) return bptr[(size_t)(kt_of(min(s * kT + g / kGroups, ntile - 1)) * kGroups + g % kGroups) * 256];
        else return bptr[(size_t)(s * kGroups + g) * 256];
    };
#pragma unroll
    for (int g = 0; g < kSet; ++g) breg[0][g] = fragment(kBurst ? 0 : rot, g);
    f32x16 acc[kBlocks];
    float ssq[kBlocks];
#pragma unroll
    for (int b = 0; b < kBlocks; ++b) {
        acc[b] = f32x16{0};
        ssq[b] = 0.0f;
    }
    // The A fragments of group g+1 are read from LDS before the matrix steps of group g are issued:
    // a wave is alone on its SIMD, so nothing else would cover the LDS round trip of each group.
    // The first kCount groups of a stage with the fragments bf; those of stage `sn` (without bursts: of k-tile `sn`) go to bnext, or into each group's
    // registers as it is done.
    auto k_stage = [&](const char* st, int sn, auto refill, auto count, u32x4 (&bf)[kSet], [[maybe_unused]] u32x4 (&bnext)[kSet]) {
        constexpr int kCount = decltype(count)::value;
        if constexpr (kBurst && decltype(refill)::value) {
#pragma unroll
            for (int g = 0; g < kSet; ++g) bnext[g] = fragment(sn, g);
            __builtin_amdgcn_sched_barrier(0);
        }
        u32x4 a[2][kBlocks];
        auto read_a = [&](int g, u32x4* dst) {
#pragma unroll
            for (int b = 0; b < kBlocks; ++b)
                dst[b] = *reinterpret_cast<const u32x4*>(st + (g / kGroups) * kTileOfRows + b * 32 * kTileBytes + (y16 ^ ((g % kGroups) << 5)));
        };
        read_a(0, a[0]);
#pragma unroll
        for (int g = 0; g < kCount; ++g) {
            u32x4* cur = a[g & 1];
            if (g + 1 < kCount) read_a(g + 1, a[(g + 1) & 1]);       // (two groups ahead: measured, no further gain)
#pragma unroll
            for (int b = 0; b < kBlocks; ++b) acc[b] = mma_k16<DT>(bf[g], cur[b], acc[b]);
            if ((g & 3) == wave_u && half_u == 0) {   // this wave's share of the sums of squares (the waves of half 0 cover every chunk)
#pragma unroll
                for (int b = 0; b < kBlocks; ++b) ssq[b] = chunk_sumsq<DT>(cur[b], ssq[b]);
            }
            if (!kBurst && decltype(refill)::value) bf[g] = fragment(sn, g);
        }
    };
    auto stage = [&](int s) { return ring + (s % kStages) * kStageBytes + a_base; };
    using Whole = std::integral_constant<int, kSet>;
    auto step = [&](int s, u32x4 (&bf)[kSet], u32x4 (&bnext)[kSet]) {
        ring_barrier();
        TIDE_STAMP();
        k_stage(stage(s), kBurst ? s + 1 : kt_of(s + 1), std::true_type{}, Whole{}, bf, bnext);
    };
    auto last_step = [&](u32x4 (&bf)[kSet]) {
        ring_barrier();
        TIDE_STAMP();
        if (kT > 1 && ntile % kT) k_stage(stage(nstage - 1), 0, std::false_type{}, std::integral_constant<int, kGroups>{}, bf, bf);
        else k_stage(stage(nstage - 1), 0, std::false_type{}, Whole{}, bf, bf);
        TIDE_STAMP();
    };
    if constexpr (kBurst) {
        int s = 0;
        for (; s + 2 < nstage; s += 2) {
            step(s, breg[0], breg[1]);
            step(s + 1, breg[1], breg[0]);
        }
        if (s + 1 < nstage) {
            step(s, breg[0], breg[1]);
            last_step(breg[1]);
        } else {
            last_step(breg[0]);
        }
    } else {
        for (int s = 0; s + 1 < nstage; ++s) step(s, breg[0], breg[0]);
        last_step(breg[0]);
    }

    if constexpr (kHalves == 2) ecols = fetch_ecols();
    // ---- row sums of squares: lanes l and l^32 hold the two chunk phases; the 4 waves the rest
#pragma unroll
    for (int b = 0; b < kBlocks; ++b) {
        const float s2 = ssq[b] + __shfl_xor(ssq[b], 32, kWave);
        if (lane < 32 && half == 0) ss_part[cw * kRowsM + 32 * b + lane] = s2;
    }
    __syncthreads();
    TIDE_STAMP();
    // every lane owns one row per block: its 1/rms from the four waves' partial sums, then the block's
    // 16 columns inside the lane
#pragma unroll
    for (int b = 0; b < kBlocks; ++b) {
        const int row = 32 * b + (lane & 31);
        const float ss = (ss_part[row] + ss_part[kRowsM + row]) + (ss_part[2 * kRowsM + row] + ss_part[3 * kRowsM + row]);
        const float z = router_epilogue_row(acc[b], kNegLog2e * inv_rms_f32(ss, p.inv_d, p.eps), ecols);
        if (lane < 32) z_part[wave * kRowsM + row] = z;
    }
    TIDE_STAMP();
    __syncthreads();
    TIDE_STAMP();
    if (tid < kRowsM) {
        const int t = row0 + tid;
        if (t < p.T) {
            float zsum = (z_part[tid] + z_part[kRowsM + tid]) + (z_part[2 * kRowsM + tid] + z_part[3 * kRowsM + tid]);
            if constexpr (kHalves == 2)
                zsum += (z_part[4 * kRowsM + tid] + z_part[5 * kRowsM + tid]) + (z_part[6 * kRowsM + tid] + z_part[7 * kRowsM + tid]);
            emit_router_result(p, c, t, p.tab.b2[c] + zsum);
        }
    }
#ifdef TIDE_TILE_TIMELINE
    __builtin_amdgcn_s_waitcnt(0);
    TIDE_STAMP();
#endif
}

}  // namespace tide
