// Prefill kernels, split-k form: the streaming computation of prefill_dma_kernel.hpp (paper
// Eq. (2), Sec. 3.4 kernel 1, Fig. 1 inference step 3) for batches with far fewer row tiles
// than the chip has CUs -- a decode step (Sec. 3.3: one or a few tokens per sequence), or the
// router call a serving loop makes at ONE checkpoint layer on a small batch.
//
// Why another form.  With fewer tiles than CUs the streaming kernel cuts tiles into pieces of
// fewer rows, but every piece still walks the whole hidden dimension against the whole W1' of
// its checkpoint: the call takes as long as one wave needs for d/16 dependent matrix steps
// (about 20 us at d = 4096, whatever the batch).  Here the k range of a tile is cut instead:
// workgroup (tile, slice) multiplies the tile's rows by 1/S of W1' and leaves its 128 partial
// sums per row, and its share of the rows' sums of squares, in the workspace; a second, small
// launch adds the S partial results of every 32-row block in a fixed order and runs the router
// epilogue and the earliest-exit report on them.  The dependent chain is S times shorter, and the
// matrix cores do the contraction, so the same pair serves 1 row and 2,000.
// Two launches, not one with a "last workgroup finishes" hand-over: that was built and measured
// -- the finishing workgroup has to read the partial results with device-scope loads (they come
// from other XCDs within the same launch), 8 bytes at a time past every cache, and at 128 rows and
// 8 slices that alone took longer (24 us a call) than the second launch costs (13 us a call).
// The price of the form is the partial results -- 16 KiB per workgroup and 32-row block, written
// once and read once -- which is why it stops where the tiles are many.  Tile height (32, 64 or
// 128 rows) and S (2, 4 or 8) are the host's choice per call: short tiles and many slices while
// the workgroups fit the chip once, fewer slices and taller tiles beyond.
// Every storage type (fp32 rows as two bf16 terms, as in the streaming kernel), d a multiple of
// 128 (kRagged: any rows of whole 16-byte chunks, zeros fetched beyond their end); at bottleneck width 256 each 128-column half of a tile is a workgroup of its own in the
// first launch.
#pragma once
#include <type_traits>

#include "device_utils.hpp"
#include "prefill_dma_kernel.hpp"

namespace tide {

constexpr int kFinishThreads = 256;

// The arguments that a launch of the pair needs before its first load, as scalars in front of the parameter block: the first 14 dwords of scalar arguments are
// in registers when a wave starts (the compiler's kernarg preload, see build.py), where the block is a round trip of some 0.2 us away.  What is needed later is fetched while the first loads are
// under way.  us, before / after: C = 1, T = 3000, d = 4096 13.3 / 12.8, T = 1000 8.7 / 8.1, C = 8, T = 200, d = 2048 8.3 / 7.9, T = 322, d = 4096 13.5 / 13.0 (without the preload 13.4).
struct SplitkTiling {          // 64 bits
    uint32_t total_tiles, tiles_per_ckpt, slices, stages, halves, deal_out, shared_lines;
    static constexpr uint32_t kMostTiles = (1 << 20) - 1, kMostSlices = 15, kMostStages = 15;      // what the fields hold
    __host__ __device__ static uint64_t pack(const PrefillParams& p) {
        return (uint64_t)(uint32_t)p.total_tiles | (uint64_t)(uint32_t)p.tiles_per_ckpt << 20 | (uint64_t)(uint32_t)p.k_slices << 40 | (uint64_t)(uint32_t)p.ring_stages << 44 |
               (uint64_t)(p.b > kBottleneck) << 48 | (uint64_t)(p.deal_out != 0) << 49 | (uint64_t)(p.shared_lines != 0) << 50;
    }
    __device__ static SplitkTiling unpack(uint64_t v) {
        const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
        return SplitkTiling{lo & 0xfffff, (uint32_t)(v >> 20) & 0xfffff, hi >> 8 & 15, hi >> 12 & 15, 1 + (hi >> 16 & 1), hi >> 17 & 1, hi >> 18 & 1};
    }
};
constexpr int kSplitkMaxS = 8;           // most workgroups that share a tile's k range (the single-launch form unrolls over them)

template <int kBlocks> constexpr int splitk_lds_bytes(int stages) { return stages * kBlocks * 32 * kTileBytes; }   // the ring
// floats a workgroup leaves in p.zpart: kBlocks*32 rows x 128 columns, in the order
// [consumer wave][block][register quad][lane][4] -- every store instruction of a wave is 1 KiB
// contiguous, and a lane of the second launch reads back the registers of its own position.
template <int kBlocks> constexpr int splitk_part_floats() { return kBlocks * 32 * kBottleneck; }

// What bounds the pair (C = 1, T = 3000, bf16, d = 4096: 14.4 us as it was, of which the second launch 4.4): a CU takes 22-28 bytes a
// cycle from beyond its own caches, rows and W1' alike, so bytes per CU set the pace of the first launch; rows and matrix steps have to overlap
// for that, and a wave alone on its SIMD takes some eight cycles for every dependent instruction.  Hence
//   - two consumer waves per SIMD, each one half of every k-tile; the two of a column block exchange halves of their accumulators at the end;
//   - up to eight k-tiles in the ring, four in flight (a producer that asks for all eight at once is held up 3.3 us in doing so and hands
//     the first one over at 3.5 us instead of 1.5);
//   - in both launches the first kernel arguments in registers and the rest in one round trip, divisions by multiplication, and in the second one 32-bit offsets, no load
//     under a condition and vector-ALU exchanges.
// us per call, before / after: 14.7 / 13.5 at C = 1, T = 3000; 14.0 / 13.5 at C = 8, T = 322; 10.5 / 9.3 at C = 1, T = 1000; fp32, C = 1, T = 3000 24.8 / 23.3;
// width 256, C = 8, T = 200 14.3 / 13.4.  (Rotating the k order of a slice from tile to tile: 0.3 us slower; channels are hashed.)
// The one-launch form keeps one wave per SIMD and four k-tiles.
constexpr int splitk_kwaves(bool fused) { return fused ? 1 : 2; }
constexpr int splitk_producers(bool fused) { return fused ? kDmaProducers : 4; }
constexpr int splitk_threads(bool fused) { return (splitk_kwaves(fused) * kDmaConsumers + splitk_producers(fused)) * kWave; }   // 384 / 768
constexpr int kSplitkMaxStages = 8;     // k-tiles of rows in the ring at most (of which four in flight)

// First launch: item = (tile * halves + half) * p.k_slices + slice (XCD-contiguous or dealt out, below); tiles of kBlocks*32 rows,
// checkpoint-major (p.tiles_per_ckpt per checkpoint); half = which 128 columns of the bottleneck
// (halves = 2 at width 256, else 1); slice s covers k-tiles [s*n/S, (s+1)*n/S) of the n = dpad/128
// k-tiles of a row (S <= n, so every slice has at least one).
// kFused (32-row tiles, widths 64 / 128, at most as many tiles as the scratch memory has counters): ONE launch.  Every
// workgroup leaves its partial results with device-scope stores -- only the register quads that hold rows in use: a
// decode step of up to 8 rows per checkpoint writes 4 KiB per workgroup instead of 16 -- and ticks the tile's counter;
// the workgroup that ticks last adds the S partial results in ascending slice order (its own included: the result does
// not depend on who is last) and finishes the router.  An earlier version of this hand-over read whole 16 KiB blocks,
// 8 bytes at a time, and lost to the second launch; with the rows in use only it wins at decode sizes (see the host's
// choice).  Ordering is by completion, as in the latency kernel (device_utils.hpp: stage_store / last_arrival).
// (fp32: 175 registers since its first arguments are scalars, 156 before: one workgroup per CU instead of two where a forced call or other work asks for two.  Held to three
// waves per SIMD it spills six and is 5 % slower, up to 18; as it is it is 5 % faster than with 156, us, 156 / 175 / held: C = 29, T = 8, d = 4096 15.8 / 15.3 / 16.5, C = 32, T = 16,
// d = 2048 12.65 / 11.3 / 12.75, and forced on more workgroups than CUs, C = 8, T = 200, d = 4096, 29.3 / 27.4 / 27.5.)
template <int DT, int kBlocks, bool kFused = false, bool kRagged = false>
__global__ __launch_bounds__(splitk_threads(kFused), 1) void tide_prefill_splitk_kernel(
    const char* hidden, const u32x4* packed, int64_t ckpt_stride_bytes, int64_t row_stride_bytes, uint64_t tiling, uint32_t by_slices_m, uint32_t by_tiles_m,
    int T, int d, const PrefillParams p) {
    static_assert(!kFused || kBlocks == 1, "the single-launch form has 32-row tiles");
    typedef __attribute__((address_space(3))) char lds_char;
    typedef __attribute__((address_space(1))) const char glb_char;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr int kRowsM = kBlocks * 32;
    constexpr int kStageBytes = kRowsM * kTileBytes;
    constexpr int kInstrPerProducer = kRowsM / 4 / splitk_producers(kFused);   // one transfer = 4 rows x 256 B
    constexpr int kKW = splitk_kwaves(kFused), kConsumers = kKW * kDmaConsumers;
    // k-tiles of W1' a consumer keeps in flight: two while the registers hold them.  (fp32, 64 rows: one, 96 registers instead of 145, us, two / one: in several
    // rounds C = 1, d = 8192, T = 4500 113.8 / 108.0, C = 6, d = 5120, T = 400, width 256 50.0 / 46.8; level in one round.)
    constexpr int kPre = kBlocks == 4 || (kBlocks == 2 && DT == kF32) ? 1 : 2;
    constexpr int kPartFloats = splitk_part_floats<kBlocks>();
    char* ring = smem;
    const SplitkTiling tl = SplitkTiling::unpack(tiling);
    const FastDiv by_slices{tl.slices, by_slices_m}, by_tiles{tl.tiles_per_ckpt, by_tiles_m};
    const int dpad = (d + 127) & ~127;                           // rows of the packed weights

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int S = (int)tl.slices, stages = (int)tl.stages, halves = (int)tl.halves;
    // XCD x (workgroup id mod 8) takes the x-th eighth of the tile-major list: a tile's partial results come from one XCD, and the
    // second launch, cut the same way, finds them in that XCD's L2 (dealt out round-robin, the slices of a tile were on eight XCDs;
    // us per call: 17.0 -> 15.3 at C = 8, T = 322, d = 4096, 16.9 -> 15.5 at C = 1, T = 3000, 18.8 -> 17.2 at 4096; width 256, C = 8, T = 200 18.8 -> 15.5).
    // Every XCD then reads the whole W1' of its tiles: few tiles of long rows are dealt out instead (p.deal_out, see deals_out in tide_route.hip),
    // and so is the one-launch form, which hands over past every cache (C = 4, T = 16, bf16: 13.0 -> 12.3 at d = 12288, 15.5 -> 13.7 at 16384).
    const int items = (int)tl.total_tiles * halves * S, per_xcd = (items + 7) >> 3;
    const bool dealt = kFused || tl.deal_out;
    const int item = dealt ? (int)blockIdx.x : (int)((blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3));
    if (item >= items || (!dealt && (int)(blockIdx.x >> 3) >= per_xcd)) return;
    const int th = by_slices(item), slice = item - th * S;
    const int tile = halves == 2 ? th >> 1 : th, half = th - tile * halves;
    const int ntile = dpad * Storage<DT>::kBytes / kTileBytes;
    const int kt0 = by_slices(slice * ntile), nk = by_slices((slice + 1) * ntile) - kt0;
    const int c = by_tiles(tile);
    const int row0 = (tile - c * (int)tl.tiles_per_ckpt) * kRowsM;
    const int cb = wave & 3;                                       // a consumer's column block

    if (wave >= kConsumers) {
        // ------------------------------------------------------------------ producers
        const int pw = wave - kConsumers;
        const int rl = lane >> 4, slot = lane & 15;
        const char* base = hidden + (int64_t)c * ckpt_stride_bytes + (int64_t)kt0 * kTileBytes;
        const char* gp[kInstrPerProducer];
        const int row_bytes = d * Storage<DT>::kBytes, whole = row_bytes / kTileBytes;   // kRagged: k-tiles from `whole` on reach beyond the rows' end
#pragma unroll
        for (int i = 0; i < kInstrPerProducer; ++i) {
            const int row = (pw * kInstrPerProducer + i) * 4 + rl;          // row within the tile
            int r = row0 + row;
            r = r < T ? r : T - 1;                                      // ragged tail: re-read the last row
            gp[i] = base + (int64_t)r * row_stride_bytes + ((slot ^ (row & 15)) << 4);
        }
        int issued = 0, slot_in = 0;
        auto issue_next = [&]() {
            if (issued >= nk) return;
            char* dst = ring + slot_in * kStageBytes;
            slot_in = slot_in + 1 == stages ? 0 : slot_in + 1;
            if (kRagged && kt0 + issued >= whole) {
#pragma unroll
                for (int i = 0; i < kInstrPerProducer; ++i) {
                    const int row = (pw * kInstrPerProducer + i) * 4 + rl;
                    const bool inside = (kt0 + issued) * kTileBytes + ((slot ^ (row & 15)) << 4) < row_bytes;
                    __builtin_amdgcn_global_load_lds((glb_char*)(inside ? gp[i] + (int64_t)issued * kTileBytes : reinterpret_cast<const char*>(g_zeros)),
                                                     (lds_char*)(dst + (pw * kInstrPerProducer + i) * 1024), 16, 0, 0);
                }
            } else {
                row_transfers<kRagged>(tl.shared_lines, [&](auto policy) {
#pragma unroll
                    for (int i = 0; i < kInstrPerProducer; ++i)
                        __builtin_amdgcn_global_load_lds((glb_char*)(gp[i] + (int64_t)issued * kTileBytes),
                                                         (lds_char*)(dst + (pw * kInstrPerProducer + i) * 1024), 16, 0, decltype(policy)::value);
                });
            }
            ++issued;
        };
        // Four stages in flight.  (More at the start hold the wave up in issuing them, and the first one is handed over late.)
        for (int s = 0; s < kDmaStages; ++s) issue_next();
        for (int k = 0; k < nk; ++k) {
            // stage k has landed once only the transfers of the younger stages are outstanding
            // (every stage is kInstrPerProducer transfers; loads complete in issue order)
            // -- at most three: four are requested at the start and one more per stage handed over
            const int younger = issued - k - 1;
            static_assert((kDmaStages - 1) * kInstrPerProducer < 64, "the wave's load counter");
            if (younger >= 3) __builtin_amdgcn_s_waitcnt(vmcnt_imm(3 * kInstrPerProducer));
            else if (younger == 2) __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * kInstrPerProducer));
            else if (younger == 1) __builtin_amdgcn_s_waitcnt(vmcnt_imm(kInstrPerProducer));
            else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
            const bool fresh = issued < stages;    // a slot that no stage has used yet: no need to wait for the consumers
            if (fresh) issue_next();
            ring_barrier();                        // stage k handed over; the consumers are done with stage k-1
            if (!fresh && k > 0) issue_next();     // ... whose slot takes the next one
        }
        if constexpr (kKW == 2) {                  // the two barriers of the consumers' exchange
            ring_barrier();
            ring_barrier();
        }
    } else {
        // ------------------------------------------------------------------ consumers
        const int wave_u = __builtin_amdgcn_readfirstlane(cb);       // uniform: branches on it are scalar
        const int kh = kKW == 2 ? __builtin_amdgcn_readfirstlane(wave >> 2) : 0;   // this wave's half of every k-tile
        const int r = lane & 31;
        const int a_base = r * kTileBytes;
        const int y16 = (((lane >> 5) ^ (r & 15)) << 4) ^ (kh << 7);   // see prefill_dma_kernel.hpp; a half k-tile is 128 bytes of a row
        const size_t ckpt_chunks = (size_t)dpad * kBottleneck / Storage<DT>::kElems;
        constexpr int kGroups = Compute<DT>::kMmaGroups / kKW, kPlanes = Compute<DT>::kPlanes;   // 16-k groups of a k-tile that this wave takes
        constexpr int kFrags = kGroups * kPlanes;                    // their W1' fragments
        const u32x4* bptr = packed + ((size_t)c * halves + half) * ckpt_chunks + (size_t)(kh * kGroups) * 256 + cb * 64 + lane;
        const size_t plane_chunks = (size_t)dpad * 16;                // fp32 rows: the hi and the mid plane of W1'
        const int yf16 = ((((lane >> 5) << 1) ^ (r & 15)) << 4) ^ (kh << 7);       // fp32 rows: see prefill_dma_kernel.hpp
        auto b_fragment = [&](int kt, int g, int pl) { return bptr[pl * plane_chunks + (size_t)(kt * Compute<DT>::kMmaGroups + g) * 256]; };
        // W1' fragments of kPre k-tiles in flight: with few k-tiles per workgroup nothing else hides
        // the L2 round trip.  Slot j holds k-tile k with k % kPre == j.
        u32x4 breg[kPre][kFrags];                                    // [g * kPlanes + plane]
#pragma unroll
        for (int j = 0; j < kPre; ++j) {
            const int kt = kt0 + (j < nk ? j : nk - 1);
#pragma unroll
            for (int g = 0; g < kGroups; ++g)
#pragma unroll
                for (int pl = 0; pl < kPlanes; ++pl) breg[j][g * kPlanes + pl] = b_fragment(kt, g, pl);
        }
        if constexpr (!kFused) asm volatile("" ::"s"(p.zpart), "s"(p.sspart));      // fetched while the first loads are under way
        f32x16 acc[kBlocks];
        float ssq[kBlocks];
#pragma unroll
        for (int b = 0; b < kBlocks; ++b) {
            acc[b] = f32x16{0};
            ssq[b] = 0.0f;
        }
        // 16-bit rows: the A fragments of a group are read from LDS kAhead groups before its matrix steps are issued: the two consumer waves of
        // a SIMD (the one-launch form: the only one) leave the barrier together, so nothing else covers the LDS round trip, and the fewer blocks
        // a tile has the fewer matrix steps there are per group to cover it with.  128 rows have registers for one group.
        constexpr int kAhead = kBlocks >= 4 ? 1 : kBlocks == 2 ? 2 : 4;
        auto read_a = [&](const char* st, int g, u32x4* dst) {
#pragma unroll
            for (int b = 0; b < kBlocks; ++b)
                dst[b] = *reinterpret_cast<const u32x4*>(st + b * 32 * kTileBytes + (y16 ^ (g << 5)));
        };
        auto k_tile = [&](const char* st, u32x4 (&bf)[kFrags], int kn, auto refill) {
            [[maybe_unused]] u32x4 a16[kAhead + 1][kBlocks];
#pragma unroll
            for (int g = 0; g < kGroups; ++g) {
                if constexpr (DT == kF32) {
                    // 16 k values = chunks 4g+2h and 4g+2h+1 of the row (4 fp32 each), each value split
                    // into two bf16 terms (device_utils.hpp); three matrix steps per group
                    u32x4 ah[kBlocks], am[kBlocks];
                    float sq[kBlocks];
#pragma unroll
                    for (int b = 0; b < kBlocks; ++b) {
                        const char* src = st + b * 32 * kTileBytes;
                        const u32x4 c0 = *reinterpret_cast<const u32x4*>(src + (yf16 ^ (g << 6)));
                        const u32x4 c1 = *reinterpret_cast<const u32x4*>(src + (yf16 ^ (g << 6) ^ 16));
                        float x[8] = {__uint_as_float(c0.x), __uint_as_float(c0.y), __uint_as_float(c0.z), __uint_as_float(c0.w),
                                      __uint_as_float(c1.x), __uint_as_float(c1.y), __uint_as_float(c1.z), __uint_as_float(c1.w)};
                        __bf16 hi[8], mid[8];
                        split_bf16(x, 8, hi, mid);
                        bf16x8 h8, m8;
#pragma unroll
                        for (int e = 0; e < 8; ++e) { h8[e] = hi[e]; m8[e] = mid[e]; }
                        ah[b] = __builtin_bit_cast(u32x4, h8);
                        am[b] = __builtin_bit_cast(u32x4, m8);
                        sq[b] = chunk_sumsq<kF32>(c1, chunk_sumsq<kF32>(c0, 0.0f));
                    }
#pragma unroll
                    for (int b = 0; b < kBlocks; ++b) acc[b] = mma_k16_split(ah[b], am[b], bf[2 * g], bf[2 * g + 1], acc[b]);
#pragma unroll
                    for (int b = 0; b < kBlocks; ++b) ssq[b] += kh * kGroups + g == wave_u ? sq[b] : 0.0f;   // this wave's share of the sums of squares
                } else {
                    if (g == 0) {
#pragma unroll
                        for (int j = 0; j < kAhead; ++j) read_a(st, j, a16[j]);
                    }
                    u32x4* a = a16[g % (kAhead + 1)];
                    if (g + kAhead < kGroups) read_a(st, g + kAhead, a16[(g + kAhead) % (kAhead + 1)]);
#pragma unroll
                    for (int b = 0; b < kBlocks; ++b) acc[b] = mma_k16<DT>(a[b], bf[g], acc[b]);
                    if ((g & 3) == wave_u) {           // this wave's share of the sums of squares
#pragma unroll
                        for (int b = 0; b < kBlocks; ++b) ssq[b] = chunk_sumsq<DT>(a[b], ssq[b]);
                    }
                }
                if (decltype(refill)::value) {
#pragma unroll
                    for (int pl = 0; pl < kPlanes; ++pl) bf[g * kPlanes + pl] = b_fragment(kn, g, pl);
                }
            }
        };
        int k = 0, slot_out = 0;
        auto next_stage = [&]() {
            const char* st = ring + slot_out * kStageBytes + a_base;
            slot_out = slot_out + 1 == stages ? 0 : slot_out + 1;
            return st;
        };
        for (; k + 2 * kPre <= nk; k += kPre) {    // steady state: every k-tile refills its slot
#pragma unroll
            for (int j = 0; j < kPre; ++j) {
                ring_barrier();
                k_tile(next_stage(), breg[j], kt0 + k + j + kPre, std::true_type{});
            }
        }
        // One to 2 kPre - 1 k-tiles are left.  Each count is a straight line of its own: with a test per k-tile the accumulators lived in two register sets
        // at every join (fp32, 64 rows: 168 and one spilled, now 145 with two k-tiles in flight; 16 bits, 32 rows 110 / 93; a few-tile call 2-4 % faster, us:
        // bf16, C = 5, T = 100, d = 4096 9.1 / 8.5, C = 1, T = 1000, d = 5120 9.9 / 9.4, one launch, C = 28, T = 8, d = 2560 10.0 / 9.7).
        if (kPre == 2 && k + 2 < nk) {             // three: the last one goes where the first of them was
            ring_barrier();
            k_tile(next_stage(), breg[0], kt0 + k + 2, std::true_type{});
            ring_barrier();
            k_tile(next_stage(), breg[kPre - 1], 0, std::false_type{});
            ring_barrier();
            k_tile(next_stage(), breg[0], 0, std::false_type{});
        } else {
            ring_barrier();
            k_tile(next_stage(), breg[0], 0, std::false_type{});
            if (kPre == 2 && k + 1 < nk) {
                ring_barrier();
                k_tile(next_stage(), breg[kPre - 1], 0, std::false_type{});
            }
        }

        float* zmine = p.zpart + (size_t)item * kPartFloats + (size_t)(cb * kBlocks) * 1024 + lane * 4;
        // ---- what this workgroup leaves behind: its accumulators as they are, and per wave one
        // partial sum of squares per row (lanes l and l^32 hold the two chunk phases)
#pragma unroll
        for (int b = 0; b < kBlocks; ++b) {
            const float s2 = ssq[b] + __shfl_xor(ssq[b], 32, kWave);
            if constexpr (kFused) {
                // register quad q holds rows 8 q + 4 (lane / 32) + (0..3): the quads below the tile's last row in use
                const int quads = (min(T - row0, 32) + 7) >> 3;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (q < quads) stage_store4(zmine + q * 256, f32x4{acc[b][4 * q], acc[b][4 * q + 1], acc[b][4 * q + 2], acc[b][4 * q + 3]});
                if (lane < 32) stage_store(p.sspart + ((size_t)item * kDmaConsumers + wave) * kRowsM + lane, s2);
            } else {
                ssq[b] = s2;
            }
        }
        if constexpr (!kFused) {
            // The two waves of a column block exchange halves of their accumulators through the ring's memory (one block: its
            // register quads 0, 1 / 2, 3; else the lower and the upper blocks); each adds and stores the half it keeps.
            constexpr int kMoved = 2 * kBlocks;                      // register quads that change hands: half of 4 kBlocks
            f32x4* ex = reinterpret_cast<f32x4*>(smem);              // [wave][kMoved][lane]
            float* ex_ss = reinterpret_cast<float*>(smem + kConsumers * kMoved * 1024);   // [wave][kBlocks][32]
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            ring_barrier();                                          // every wave is done with the ring
            auto quad = [&](int q) { return f32x4{acc[q >> 2][(q & 3) * 4], acc[q >> 2][(q & 3) * 4 + 1], acc[q >> 2][(q & 3) * 4 + 2], acc[q >> 2][(q & 3) * 4 + 3]}; };
#pragma unroll
            for (int j = 0; j < kMoved; ++j) {
                const f32x4 lo = quad(j), hi = quad(kMoved + j);
                ex[(wave * kMoved + j) * kWave + lane] = kh ? lo : hi;
            }
#pragma unroll
            for (int b = 0; b < kBlocks; ++b)
                if (lane < 32) ex_ss[(wave * kBlocks + b) * 32 + lane] = ssq[b];
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            ring_barrier();
            const int other = wave ^ 4;
#pragma unroll
            for (int j = 0; j < kMoved; ++j) {
                const f32x4 lo = quad(j), hi = quad(kMoved + j);
                const f32x4 sum = (kh ? hi : lo) + ex[(other * kMoved + j) * kWave + lane];
                *reinterpret_cast<f32x4*>(zmine + (kh * kMoved + j) * 256) = sum;
            }
#pragma unroll
            for (int b = 0; b < kBlocks; ++b)
                if (lane < 32 && 2 * b / kBlocks == kh)
                    p.sspart[((size_t)item * kDmaConsumers + cb) * kRowsM + 32 * b + lane] = ssq[b] + ex_ss[(other * kBlocks + b) * 32 + lane];
        }
    }
    if constexpr (kFused) {
        // ---- the workgroup that completes the tile's count finishes it (every wave of the workgroup takes part in
        // the barriers; the ring is no longer in use, its memory holds the exchange arrays)
        float* inv_rms = reinterpret_cast<float*>(smem);          // [32], 16-byte aligned
        float* z_part = inv_rms + 32;                             // [4][32]
        int* flag = reinterpret_cast<int*>(z_part + 4 * 32);
        stage_writes_done();
        if (!last_arrival(p.counters + tile, (uint32_t)S, flag)) return;
        const int quads = (min(T - row0, 32) + 7) >> 3;
        const size_t first_item = (size_t)tile * S;
        if (wave < kDmaConsumers) {
            // this lane's column of the second layer, fetched first so that the epilogue does not wait for it
            const int col = 32 * wave + (lane & 31);
            const float b1c = (p.b1 && col < p.b) ? p.b1[c * p.b + col] : 0.0f;
            const float w2c = col < p.b ? p.w2[c * p.b + col] : 0.0f;
            // sums of squares: lane (h, r) takes waves 2h, 2h+1 of every slice (surplus loads re-read the last slice)
            const float* sp = p.sspart + first_item * kDmaConsumers * kRowsM + (size_t)(2 * (lane >> 5)) * kRowsM + (lane & 31);
            float sa[kSplitkMaxS], sb[kSplitkMaxS];
#pragma unroll
            for (int j = 0; j < kSplitkMaxS; ++j) {
                const size_t o = (size_t)(j < S ? j : S - 1) * kDmaConsumers * kRowsM;
                sa[j] = stage_load(sp + o);
                sb[j] = stage_load(sp + o + kRowsM);
            }
            // this wave's 32 columns: the S partial accumulators of its lane position, all loads in flight; one
            // straight-line version per number of register quads in use (a branch around a load makes the compiler wait)
            const float* zp = p.zpart + first_item * kPartFloats + (size_t)wave * 1024 + lane * 4;
            f32x4 sum[4] = {f32x4{0}, f32x4{0}, f32x4{0}, f32x4{0}};
            auto add_slices = [&](auto quads_tag) {
                constexpr int kQ = decltype(quads_tag)::value;
                f32x4 v[kSplitkMaxS][kQ];
#pragma unroll
                for (int j = 0; j < kSplitkMaxS; ++j) {
                    const size_t o = (size_t)(j < S ? j : S - 1) * kPartFloats;
#pragma unroll
                    for (int q = 0; q < kQ; ++q) v[j][q] = stage_load4(zp + o + q * 256);
                }
#pragma unroll
                for (int j = 0; j < kSplitkMaxS; ++j) {
                    const bool keep = j < S;
#pragma unroll
                    for (int q = 0; q < kQ; ++q) sum[q] += keep ? v[j][q] : f32x4{0};
                }
            };
            switch (quads) {
            case 1: add_slices(std::integral_constant<int, 1>{}); break;
            case 2: add_slices(std::integral_constant<int, 2>{}); break;
            case 3: add_slices(std::integral_constant<int, 3>{}); break;
            default: add_slices(std::integral_constant<int, 4>{}); break;
            }
            float ss = 0.0f;
#pragma unroll
            for (int j = 0; j < kSplitkMaxS; ++j) ss += j < S ? sa[j] + sb[j] : 0.0f;
            ss += __shfl_xor(ss, 32, kWave);
            if (wave == 0 && lane < 32) inv_rms[lane] = inv_rms_f32(ss, p.inv_d, p.eps);
            __syncthreads();
            f32x16 facc[1];
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) facc[0][4 * q + e] = sum[q][e];
            router_epilogue<1>(facc, inv_rms, z_part + wave * 32, b1c, w2c, lane);
        } else {
            __syncthreads();
        }
        __syncthreads();
        if (tid == 0) __hip_atomic_store(p.counters + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // zero for the next call
        if (tid < 32) {
            const int t = row0 + tid;
            if (t < T) {
                const float z = p.tab.b2[c] + ((z_part[tid] + z_part[32 + tid]) + (z_part[64 + tid] + z_part[96 + tid]));
                emit_router_result(p, c, t, z);
            }
        }
    }
}

// Second launch: one workgroup per 8 kQ rows -- kQ register quads of a 32-row block, item = (tile * kBlocks + block) * 4 / kQ +
// group of quads -- with 4 waves per column half; wave w of a half owns its columns 32w..32w+31 as consumer wave w of the first
// launch did.  Slices are added in ascending order: the result does not depend on timing.  It is a chain of latencies (its start,
// the partial results from this XCD's L2, the epilogue, the report), so it is cut finer than the 32-row blocks of the first
// launch: an eighth of the loads per lane and a quarter of the SiLUs, which took 0.5-1 us off a call (12.5 -> 11.6 us at C = 1, T = 1024,
// 14.6 -> 13.6 at 2048, 17.4 -> 16.9 at 3000; width 256, C = 8, T = 200 21.2 -> 18.9).
template <int kBlocks, int kHalves, int kQ, int kS>
__global__ __launch_bounds__(kFinishThreads * kHalves) void tide_splitk_finish_kernel(
    const float* zpart, const float* b1, const float* w2, uint64_t tiling, uint32_t by_tiles_m, float inv_d, int T, int b, const PrefillParams p) {
    constexpr int kRows8 = 8 * kQ;
    __shared__ float z_part[4 * kHalves][kRows8];
    __shared__ float ss_part[4][kRows8];
    constexpr uint32_t kRowsM = kBlocks * 32;
    constexpr uint32_t kPartBytes = splitk_part_floats<kBlocks>() * sizeof(float);
    const SplitkTiling tl = SplitkTiling::unpack(tiling);
    const FastDiv by_tiles{tl.tiles_per_ckpt, by_tiles_m};
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6), half = wave >> 2, w = wave & 3;
    const uint32_t groups = tl.total_tiles * kBlocks * (4 / kQ), per_xcd = (groups + 7) >> 3;
    const uint32_t item = tl.deal_out ? blockIdx.x : (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);           // (see the first launch)
    if (item >= groups || (!tl.deal_out && (blockIdx.x >> 3) >= per_xcd)) return;
    const uint32_t quad = (item % (4 / kQ)) * kQ, tb = item / (4 / kQ);
    const uint32_t tile = tb / kBlocks, blk = tb - tile * kBlocks;
    const uint32_t c = by_tiles((int)tile);
    const uint32_t row0 = (tile - c * tl.tiles_per_ckpt) * kRowsM + 32 * blk + 8 * quad;
    if (row0 >= (uint32_t)T) return;             // padding rows only
    const uint32_t S = tl.slices;                 // at most kS
    // partial accumulators: rows 8 q + 4 (lane / 32) + (0..3) of the block per quad, one column per lane; all slices' loads in
    // flight (a surplus load re-reads the last slice).  Offsets into the partial results have 32 bits: they are 512 MiB at most.
    const char* zp = reinterpret_cast<const char*>(zpart) + ((tile * kHalves + half) * S * kPartBytes + (w * kBlocks + blk) * 4096 + quad * 1024);
    f32x4 v[kS][kQ];
#pragma unroll
    for (uint32_t j = 0; j < kS; ++j) {
#pragma unroll
        for (int q = 0; q < kQ; ++q) v[j][q] = *reinterpret_cast<const f32x4*>(zp + (uint32_t)(q * 1024 + lane * 16));
        if (j + 1 < kS) zp += j + 1 < S ? kPartBytes : 0;
    }
    // partial sums of squares (those of column half 0; every half computed the same ones): thread (row, slice, column block of the first launch)
    const bool squares = kHalves == 1 || half == 0;
    const uint32_t sl = tid >> 5;
    float ss[kQ];
    if (squares) {
        const char* sp = reinterpret_cast<const char*>(zpart) + (size_t)tl.total_tiles * kHalves * S * kPartBytes +
                         ((tile * kHalves * S + (sl < S ? sl : S - 1)) * kDmaConsumers + ((tid >> 3) & 3)) * (kRowsM * 4) + (32 * blk + 8 * quad + (tid & 7)) * 4;
#pragma unroll
        for (int q = 0; q < kQ; ++q) ss[q] = *reinterpret_cast<const float*>(sp + 32 * q);
    }
    // this lane's column of the second layer (columns at and beyond the bottleneck width are zero padding: their w2 is zero), branch-free
    const uint32_t col = kBottleneck * half + 32 * w + (lane & 31), at = c * b + (col < (uint32_t)b ? col : 0);
    float b1c = (b1 ? b1 : w2)[at], w2c = w2[at];
    if (!b1) b1c = 0.0f;
    if (col >= (uint32_t)b) w2c = 0.0f;
    // what the end needs, fetched while the partial results are under way
    const float b2c = p.tab.b2[c], thr = p.tab.thr_logit[c];
    TIDE_FETCH_ARGS8(p.eps, p.C, p.logits, p.exit_layer, p.arrive, p.fire_mask, b2c, thr);
    if (squares) {
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
            const float t = add_xor<32>(add_xor<16>(add_xor<8>(sl < S ? ss[q] : 0.0f)));
            if (lane < 8) ss_part[w][8 * q + lane] = t;
        }
    }
    f32x4 sum[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
        sum[q] = v[0][q];
#pragma unroll
        for (uint32_t j = 1; j < kS; ++j) sum[q] += j < S ? v[j][q] : f32x4{0, 0, 0, 0};
    }
    __syncthreads();
    const int h = lane >> 5;
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
        float x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = 8 * q + 4 * h + e;
            const float inv = inv_rms_f32((ss_part[0][row] + ss_part[1][row]) + (ss_part[2][row] + ss_part[3][row]), inv_d, p.eps);
            x[e] = w2c * silu_f32(fmaf(inv, sum[q][e], b1c));
        }
        const float total = reduce_scatter4(x, lane);     // of row 4 h + 2 (bit 3 of the lane) + (bit 2), in every lane of it
        if ((lane & 19) == 0) z_part[wave][8 * q + 4 * h + ((lane >> 3) & 1) * 2 + ((lane >> 2) & 1)] = total;
    }
    __syncthreads();
    if (tid < kRows8) {
        const int t = row0 + tid;
        if (t < T) {
            float zsum = (z_part[0][tid] + z_part[1][tid]) + (z_part[2][tid] + z_part[3][tid]);
            if constexpr (kHalves == 2) zsum += (z_part[4][tid] + z_part[5][tid]) + (z_part[6][tid] + z_part[7][tid]);
            emit_router_result(p, c, t, b2c + zsum, thr);
        }
    }
}

}  // namespace tide
