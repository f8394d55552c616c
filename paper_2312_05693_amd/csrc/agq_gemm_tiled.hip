// Tiled int8-MFMA kernel of the quantized linear layer for many tokens (the
// prefill regime, bound by the matrix cores).
//
// Workgroup tile 128 (tokens) x 128 (output channels), K step 128, four
// wavefronts as 2 (tokens) x 2 (channels): each owns 64 x 64 as 2 x 2 MFMA tiles
// of 32 x 32 (v_mfma_i32_32x32x32_i8, 64 accumulator registers per lane).  Two
// workgroups share a CU, one wavefront of each per SIMD: a workgroup barrier (one
// per K step), a prologue or an epilogue stalls only one of the two wavefronts
// that feed a matrix core.  The 32 x 32 x 32 form is used because back-to-back
// 16 x 16 x 64 MFMAs of one wavefront keep the matrix core only 55 % busy.
// Three variants serve calls with few tiles: 64-token tiles (NI == 1), the same with
// the K steps of a tile shared by two wavefront groups (KG == 2), and a split of
// K over workgroups (SPLIT), all described at the kernel.
//
//   activation codes: int8, already laid out in MFMA operand order by the
//     pre-pass (16 KiB per 128-token tile and K step, see agq_quant.hip), copied
//     HBM/L2 -> LDS by direct global-to-LDS loads (no registers in between,
//     contiguous 1 KiB per instruction), three stages deep.  A fragment read is
//     one conflict-free ds_read_b128 at lane * 16.
//   weights: the packed 4-bit blob is copied the same way (16 bytes per lane,
//     512-byte contiguous runs); a wavefront reads its 64 channels back once per
//     step and widens them to int8 in registers: three bit operations per eight
//     weights.  The nibbles cross HBM, L2 and LDS at half the bytes of int8.  A
//     lane addresses the blob's 16-row chunks so that it receives the operand
//     of a 32-row MFMA: low nibbles feed k-block t, high nibbles k-block t + 2.
//   No load in the main loop returns to registers, so the only waits on vector
//   memory are the ones written here: loads return in order, every step issues
//   as many per wavefront, and a step waits until at most those of the step two
//   ahead are still in flight (copies start three steps ahead; the fragments of the
//   step being multiplied are already in registers, so three stages suffice).
//
// The weight fragment is the MFMA's first operand and the activation the second:
// a lane then holds four consecutive output channels of one token.  The
// epilogue dequantizes in registers, transposes through LDS (free by then) and
// stores whole 128-byte rows, 16 bytes per lane.
#include "../../include/agq.h"
#include "agq_device.h"
#include "agq_internal.h"

#include <type_traits>

typedef unsigned int agq_u4 __attribute__((ext_vector_type(4)));
typedef int agq_v16i __attribute__((ext_vector_type(16)));

namespace {

constexpr int BM = 128, BN = 128, BK = 128;
constexpr int kThreads = 256;
constexpr int kBand = 4;                  // token tiles per band of the tile walk
constexpr int kBChunks = BN / 16;         // 8 chunks of 1 KiB per stage
constexpr int kStages = 3;
constexpr int kOutStride = 144;           // bytes per row of a wavefront's 64 x 64 fp16 output tile in LDS

constexpr int kMaxProj = 4;   // == AGQ_MAX_PROJ of the public header

// Up to four projections of the same activation share a launch (q/k/v, gate/up): one
// grid covers the tiles of all of them, which fills the chip where a single projection
// has too few tiles and saves the gaps between launches.
struct TiledProj {
    const agq_u4 *blob;
    const __half *sw;
    __half *y;
    int32_t *acc;
    const int32_t *wsum;    // per-channel weight sums (end of every blob)
    int64_t ldy;
    int N, tiles_n, start;  // start: first tile of the projection
};
struct TiledArgs {
    TiledProj proj[kMaxProj];   // projections past the last one repeat it, with no tile left for them
    const agq_u4 *xt;    // activation codes in operand order (pre-pass output)
    int M, K, KT;
    int tiles_m;
    float scale_e;
    int corr;               // unsigned activation grid: acc += corr * wsum[n]; 0 on the signed grid
    // TRIP blob: the first n_extra steps are the extra chunks of the channels with a factor;
    // trip_shift[kt] (device) is the left shift of the running accumulators after step kt
    int n_extra;
    const int32_t *trip_shift;
    // K split over `splits` workgroups per tile (few tiles, long K), steps_per_split K steps each: they
    // leave int32 partial tiles in `part`, which a second kernel adds up and dequantizes
    int splits, steps_per_split, tiles_all;
    int32_t *part;       // [tile][split][16][256 threads][4]
};

// The projection a workgroup serves is read from the argument record where it lies, in constant memory: an index
// into the by-value parameter would copy all of it to memory, and selects over its four entries took the kernel
// 160 spilled scalar registers and several hundred instructions before its first copy.
typedef const __attribute__((address_space(4))) TiledArgs TiledArgsC;
typedef const __attribute__((address_space(4))) TiledProj TiledProjC;
__device__ __forceinline__ TiledProjC *tiled_proj(const TiledArgs &a, int tile) {
    const int pj = (tile >= a.proj[1].start) + (tile >= a.proj[2].start) + (tile >= a.proj[3].start);
    return ((TiledArgsC *)__builtin_amdgcn_kernarg_segment_ptr())->proj + pj;
}

template <int N>
struct Int {
    static constexpr int value = N;
};

// TRIP: the blob and the activation stages carry extra steps in front, ordered by
// descending factor; after the last step of a factor the accumulators are shifted
// left by the difference to the next factor (Horner), so that at the end every
// extra step has been multiplied by 2^factor (Section 4.4) - exact in int32.
//
// SPLIT: with fewer tiles than the chip has workgroup slots and a long K, a tile's K steps are shared
// out over several workgroups.  Each stores its int32 accumulators as a partial tile and is done;
// split_reduce_kernel, launched behind it, adds the partial tiles up and runs the epilogue.  (One
// kernel in which the last workgroup to arrive at a tile adds the others' partial tiles was measured
// slower than no split at all: it has to read them in dependent rounds through device-scope loads,
// or with cache-wide write-backs and invalidations around them.)  An int32 sum does not depend on
// its order, so the result is the unsplit kernel's bit for bit.
//
// NI: 32-token MFMA tiles per wavefront.  2: the 128-token workgroup tile described above.  1: a 64-token
// tile (each wavefront 32 x 64, half of the MFMAs per step for two thirds of the operand bytes), for grids
// whose 128-token tiles would leave the last round of workgroups mostly empty.
//
// KG: groups of four wavefronts that share the K steps of the workgroup's tile, each with stages of its own; they meet at
// the same barriers, and at the end group 1 hands its sums to group 0 through LDS.  With one workgroup on a CU a single
// wavefront per SIMD waits at every barrier with the matrix core idle (64-token tiles, K = 11008, 100 tokens: 0.24 us a
// step, of which the MFMAs are 0.12; 0.36 with the weights from HBM); two groups take 0.36 (0.52) us for two steps.
// 128-token tiles gain nothing from it (0.29 against 0.26 us a step), nor does either from more than three stages.
template <bool TRIP, bool SPLIT, int NI, int KG>
__global__ __launch_bounds__(kThreads * KG, 2) void gemm_tiled_kernel(const TiledArgs a) {
    static_assert(NI == 2 || (NI == 1 && !SPLIT), "the partial tiles of a K split are laid out for 128 tokens");
    static_assert(KG == 1 || (KG == 2 && !SPLIT), "one kind of K split at a time");
    constexpr int BMT = NI * 64;                 // tokens per workgroup tile
    constexpr int kAChunksT = NI * 8;            // activation chunks of 1 KiB per stage
    constexpr int kStageT = (kAChunksT + kBChunks) * 1024;   // 24 KiB (16 KiB for NI == 1)
    constexpr int kNA = NI * 2;                  // activation copies per wavefront and step
    constexpr int kCopiesT = kNA + 2;
    // Three pipeline stages per K group; the epilogue reuses the first 18 NI KiB.
    __shared__ __align__(16) unsigned char lds[KG * kStages * kStageT];
    const int lane = threadIdx.x & 63;
    const int wave = (threadIdx.x >> 6) & 3;
    const int grp = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    const int tid = threadIdx.x & (kThreads - 1);        // in the K group
    const int wm = wave >> 1, wn = wave & 1;

    // XCD-aware tile order.  Consecutive workgroup ids land on different XCDs
    // (round-robin over 8), each with its own L2, so first give every XCD a
    // contiguous run of logical tile ids (the first nblk % 8 of them one more); then walk the tile grid in bands of
    // kBand token tiles, column by column, so that a run covers a compact
    // rectangle and re-reads as little of either operand as possible.
    const int nblk = gridDim.x;
    int bid = blockIdx.x;
    bid = (bid & 7) * (nblk >> 3) + min(bid & 7, nblk & 7) + (bid >> 3);
    // SPLIT: workgroups with the same K slice are neighbours (they share activation stages)
    const int split = SPLIT ? bid / a.tiles_all : 0;
    if (SPLIT) bid -= split * a.tiles_all;
    const int tile_id = bid;
    TiledProjC *const pr = tiled_proj(a, bid);
    bid -= pr->start;
    const int pN = pr->N, ptiles_n = pr->tiles_n;
    const agq_u4 *const pblob = pr->blob;
    const __half *const psw = pr->sw;
    __half *const py = pr->y;
    const int64_t pldy = pr->ldy;
    int32_t *const pacc = pr->acc;
    const int32_t *const pwsum = pr->wsum;
    const int band = bid / (kBand * ptiles_n);
    const int rows = min(kBand, a.tiles_m - band * kBand);
    const int within = bid - band * kBand * ptiles_n;
    const int tn = within / rows, tm = band * kBand + within - tn * rows;
    const int m0 = tm * BMT, n0 = tn * BN;
    const int KTfull = a.KT;
    const int kwg = SPLIT ? split * a.steps_per_split : 0;
    const int KTwg = SPLIT ? min(a.steps_per_split, KTfull - kwg) : KTfull;  // steps of this workgroup
    // KG == 2: the first half for group 0 (the extra steps, whose shifts apply to what came before them, stay together),
    // the rest for group 1.  (Two steps at least, and the extra steps are never all of them: neither group is empty.)
    const int khalf = KG == 1 ? KTwg : max((KTwg + 1) >> 1, TRIP ? a.n_extra : 0);
    const int kbeg = kwg + (grp == 1 ? khalf : 0);
    const int KT = grp == 1 ? KTwg - khalf : khalf;      // steps of this group

    // Copies of this wavefront per step: activation chunks 4 wave .. 4 wave + 3 of
    // the 16 KiB stage, and weight chunks 2 wave, 2 wave + 1.  Weight chunk c
    // serves channel group c >> 2 (64 channels), 32-channel tile (c >> 1) & 1,
    // k-blocks t = c & 1 (low nibbles) and t + 2 (high nibbles): channel l & 31
    // of the tile lives in the blob's 16-row chunk (l & 31) >> 4 at blob lane
    // (2 t + (l >> 5)) * 16 + (l & 15).
    // (NI == 1: the 64-token tile tm is half tm & 1 of the 128-token tile tm >> 1 of the pre-pass: eight
    // consecutive chunks of every stage, two per wavefront)
    const uint32_t wave_u = __builtin_amdgcn_readfirstlane((uint32_t)wave);
    const int atile = NI == 2 ? tm : tm >> 1, achunk = (NI == 2 ? 0 : (tm & 1) * 8) + (int)wave_u * kNA;
    const char *abase = reinterpret_cast<const char *>(a.xt) + (((int64_t)atile * KTfull + kbeg) * 16 + achunk) * 1024;
    const char *bbase = reinterpret_cast<const char *>(pblob) + ((int64_t)(n0 / 16) * KTfull + kbeg) * 1024;
    const uint32_t avoff = (uint32_t)lane * 16;
    uint32_t bvoff[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int c = wave * 2 + p, grp = c >> 2, j = (c >> 1) & 1, t = c & 1;
        const int chunk_row = grp * 4 + j * 2 + ((lane & 31) >> 4);
        bvoff[p] = (uint32_t)chunk_row * (uint32_t)KTfull * 1024u + (uint32_t)((2 * t + (lane >> 5)) * 16 + (lane & 15)) * 16u;
    }
    // LDS byte address (wave-uniform, kept in a scalar register) of this
    // wavefront's first activation chunk in stage 0
    const uint32_t lds_base = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) unsigned char *)lds) + grp * (kStages * kStageT);
    const uint32_t lds_a = lds_base + wave_u * (kNA * 1024), lds_b = lds_base + kAChunksT * 1024 + wave_u * 2048;
    // copy p of a step into the stage that starts `st` bytes into lds, from the step's source addresses (the
    // activation pieces of a wavefront are contiguous on both sides: one base, the piece in the offset)
    auto copy_piece = [&](auto p_tag, uint32_t st, const char *ap, const char *bp) {
        constexpr int p = decltype(p_tag)::value;
        if constexpr (p < kNA) lds_dma16_s<0, p * 1024>(avoff, ap, lds_a + st);
        else lds_dma16_s<(p - kNA) * 1024, 0>(bvoff[p - kNA], bp, lds_b + st);
    };
    auto copy_a = [&](uint32_t st, const char *ap) {
        copy_piece(Int<0>{}, st, ap, nullptr);
        copy_piece(Int<1>{}, st, ap, nullptr);
        if constexpr (kNA == 4) {
            copy_piece(Int<2>{}, st, ap, nullptr);
            copy_piece(Int<3>{}, st, ap, nullptr);
        }
    };
    auto copy_b = [&](uint32_t st, const char *bp) {
        copy_piece(Int<kNA>{}, st, nullptr, bp);
        copy_piece(Int<kNA + 1>{}, st, nullptr, bp);
    };
    // The first three steps, or all of fewer.  (Copying the last step again instead of branching: 512 tiles of one step,
    // 128 -> 8192 at 1000 tokens, 12.1 against 11.8 us with the pre-pass, of two steps 11.6 against 11.4; no
    // difference from six steps on.)
    copy_a(0, abase);
    if (KT > 1) copy_a(kStageT, abase + 16384);
    if (KT > 2) copy_a(2 * kStageT, abase + 2 * 16384);

    // per-channel scales of this lane's output columns, fetched early
    // (accumulator register 4 q + r of tile j: channel 32 j + 8 q + 4 (lane >> 5) + r)
    const int ncol = n0 + wn * 64 + (lane >> 5) * 4;
    uint2 swp[2][4];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int n = ncol + j * 32 + q * 8;
            // channels past N are never stored: clamp their addresses into the array
            const uint16_t *sp = reinterpret_cast<const uint16_t *>(psw);
            if ((pN & 3) == 0) {
                swp[j][q] = *reinterpret_cast<const uint2 *>(sp + min(n, pN - 4));   // 8-byte aligned: n % 4 == 0
            } else {
                uint32_t h[4];
                for (int r = 0; r < 4; ++r) h[r] = sp[min(n + r, pN - 1)];
                swp[j][q] = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
            }
        }

    agq_v16i acc[NI][2];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

    // Fragments of a whole step live in registers: NI * 4 activation fragments
    // (index i * 4 + t: 32-token tile i, k-block t) and four packed weight pieces.
    // Two such sets alternate: while one is multiplied, the other is filled from
    // the next step's LDS stage, so no MFMA ever waits for an LDS read it issued
    // a few instructions earlier.
    agq_u4 xa0[NI * 4], b0[4], xa1[NI * 4], b1[4];

    // One K step, software-pipelined by hand.  A wavefront issues in order, one
    // instruction every four cycles, and an MFMA waits at issue until the matrix
    // core is done with the one before it: what follows an MFMA is hidden by it up to
    // about seven instructions, and anything beyond that leaves the matrix core
    // idle.  So the other work of a step is dealt out one MFMA at a time: after each of
    // the 8 NI MFMAs at most one LDS read for the next step, one copy of the step
    // three ahead, and 4 / NI words of the weights of the next k-block widened (the first
    // k-block of the next step included, so that a step starts with an MFMA).  Nothing
    // in the steady loop branches (a branch around each copy costs more than the copies).
    // Measured against the same work in bunches behind every second MFMA (1024 tokens, one
    // workgroup per CU): 0.58 -> 0.48 us per step.  What is left is not latency: six stages instead of
    // three change nothing, while the loop without its copies takes 0.36 us and with its MFMAs alone
    // 0.31 us, at 1.6-1.75 GHz: under this load the chip runs at its power limit, so every byte moved costs time.
    const char *anext = abase + 3 * 16384, *bnext = bbase + 3 * 1024;   // sources of the step three ahead
    uint32_t rd = kStageT, fill = 0;                     // stage read from (next step), stage refilled
    constexpr int kSlots = 8 * NI;                       // MFMAs of a step
    constexpr int kReads = 4 * NI + 4;
    const agq_u4 *const rda = reinterpret_cast<const agq_u4 *>(lds + grp * (kStages * kStageT)) + lane + wm * (NI * 4 * 64);
    const agq_u4 *const rdb = reinterpret_cast<const agq_u4 *>(lds + grp * (kStages * kStageT)) + lane + (kAChunksT + wn * 4) * 64;
    agq_v4i wb[2][2];                                    // widened weights of this k-block and the next
    auto widen1 = [&](const agq_u4 (&bc)[4], int t, int d) {   // dword d (0..7) of k-block t
        const uint32_t p = bc[(d >> 2) * 2 + (t & 1)][d & 3];
        wb[t & 1][d >> 2][d & 3] = (int)(t < 2 ? ((p << 4) & 0xF0F0F0F0u) : (p & 0xF0F0F0F0u));
    };
    auto step = [&](auto copy_tag, auto next_tag, const agq_u4 (&xc)[NI * 4], const agq_u4 (&bc)[4], agq_u4 (&xn)[NI * 4], agq_u4 (&bn)[4]) {
        constexpr bool COPY = decltype(copy_tag)::value, NEXT = decltype(next_tag)::value;
        const agq_u4 *const sa = rda + rd / 16, *const sb = rdb + rd / 16;
        auto slot = [&](auto slot_tag) {
            constexpr int sl = decltype(slot_tag)::value, t = sl / (2 * NI), i = (sl - t * 2 * NI) / 2, j = sl & 1;
            if constexpr (sl < kSlots) {
                acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wb[t & 1][j], __builtin_bit_cast(agq_v4i, xc[i * 4 + t]), acc[i][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (NEXT && sl < kReads) {     // b0 b2 x.0 b1 b3 x.1 x.2 x.3
                    constexpr int h = sl / (NI + 2), q = sl - h * (NI + 2);
                    if constexpr (h < 2 && q < 2) bn[q * 2 + h] = sb[(q * 2 + h) * 64];
                    else {
                        constexpr int m = h < 2 ? h * NI + q - 2 : sl - 4;
                        xn[(m % NI) * 4 + m / NI] = sa[((m % NI) * 4 + m / NI) * 64];
                    }
                }
                constexpr int cs = NI == 2 ? sl - 3 : sl - 1;
                if constexpr (COPY && cs >= 0 && (cs & 1) == 0 && cs / 2 < kCopiesT) copy_piece(Int<cs / 2>{}, fill, anext, bnext);
                constexpr int wd = 4 / NI;               // dwords widened per slot
                constexpr int w0 = (sl - t * 2 * NI) * wd;
#pragma unroll
                for (int d = w0; d < w0 + wd; ++d) {
                    if constexpr (t < 3) widen1(bc, t + 1, d);
                    else if constexpr (NEXT) widen1(bn, 0, d);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        slot(Int<0>{}); slot(Int<1>{}); slot(Int<2>{}); slot(Int<3>{}); slot(Int<4>{}); slot(Int<5>{}); slot(Int<6>{}); slot(Int<7>{});
        slot(Int<8>{}); slot(Int<9>{}); slot(Int<10>{}); slot(Int<11>{}); slot(Int<12>{}); slot(Int<13>{}); slot(Int<14>{}); slot(Int<15>{});
        if (COPY) {
            anext += 16384;
            bnext += 1024;
            fill = fill == 2 * kStageT ? 0 : fill + kStageT;
        }
        rd = rd == 2 * kStageT ? 0 : rd + kStageT;
    };

    auto shift_acc = [&](int sh) {          // uniform
        if (sh == 0) return;
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] <<= sh;
    };

    copy_b(0, bbase);
    if (KT > 1) copy_b(kStageT, bbase + 1024);
    if (KT > 2) copy_b(2 * kStageT, bbase + 2 * 1024);
    // vmcnt(n) lgkmcnt(0): bits 3:0 and 15:14 = vmcnt, 6:4 = 7 (no wait), 11:8 = lgkmcnt
#define AGQ_WAIT(VM) __builtin_amdgcn_s_waitcnt(((VM) & 15) | (((VM) >> 4) << 14) | 0x70)
    if (KT > 2) AGQ_WAIT(2);   // steps 0 and 1 have landed (the weights of step 2 are the last two copies)
    else AGQ_WAIT(0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    {
        const agq_u4 *s0 = reinterpret_cast<const agq_u4 *>(lds + grp * (kStages * kStageT)) + lane;
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int t = 0; t < 4; ++t) xa0[i * 4 + t] = s0[((wm * NI + i) * 4 + t) * 64];
#pragma unroll
        for (int j = 0; j < 4; ++j) b0[j] = s0[(kAChunksT + wn * 4 + j) * 64];
    }
    // Between two steps: this wavefront's copies of the next step have landed (at most VM newer ones may fly: loads
    // return in order) and its reads of the stage that is refilled next have returned; then meet the others.  (Not
    // __syncthreads(), in front of which the compiler may wait for more.)
#define AGQ_MEET(VM)                              \
    asm volatile("" ::: "memory");                \
    __builtin_amdgcn_sched_barrier(0);            \
    AGQ_WAIT(VM);                                 \
    __builtin_amdgcn_s_barrier();                 \
    asm volatile("" ::: "memory");                \
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int d = 0; d < 8; ++d) widen1(b0, 0, d);
#define AGQ_SHIFT(KT_) if (TRIP && split == 0 && grp == 0 && (KT_) < a.n_extra) shift_acc(a.trip_shift[KT_]);
    // stages rotate through three, the register sets through two; the copies of the step two ahead stay in flight
    int kt = 0;
    for (; kt + 4 < KT; kt += 2) {
        AGQ_MEET(kCopiesT)
        step(std::true_type{}, std::true_type{}, xa0, b0, xa1, b1);
        AGQ_SHIFT(kt)
        AGQ_MEET(kCopiesT)
        step(std::true_type{}, std::true_type{}, xa1, b1, xa0, b0);
        AGQ_SHIFT(kt + 1)
    }
    if (kt + 3 < KT) {                                   // four steps are left, or up to three
        AGQ_MEET(kCopiesT)
        step(std::true_type{}, std::true_type{}, xa0, b0, xa1, b1);
        AGQ_SHIFT(kt)
        ++kt;
#pragma unroll
        for (int i = 0; i < NI * 4; ++i) xa0[i] = xa1[i];
#pragma unroll
        for (int i = 0; i < 4; ++i) b0[i] = b1[i];
    }
    if (kt + 1 < KT) {
        AGQ_MEET(kCopiesT)
        step(std::false_type{}, std::true_type{}, xa0, b0, xa1, b1);
        AGQ_SHIFT(kt)
        ++kt;
        if (kt + 1 < KT) {
            AGQ_MEET(0)
            step(std::false_type{}, std::true_type{}, xa1, b1, xa0, b0);
            AGQ_SHIFT(kt)
            ++kt;
        } else {
#pragma unroll
            for (int i = 0; i < NI * 4; ++i) xa0[i] = xa1[i];
#pragma unroll
            for (int i = 0; i < 4; ++i) b0[i] = b1[i];
        }
    }
    AGQ_MEET(0)
    step(std::false_type{}, std::false_type{}, xa0, b0, xa1, b1);
    AGQ_SHIFT(kt)
#undef AGQ_SHIFT
#undef AGQ_MEET
#undef AGQ_WAIT
    if (KG == 2) {
        // the groups meet once per step and once before the first one: the shorter one catches up
        for (int more = KTwg - 2 * KT; more > 0; --more) __builtin_amdgcn_s_barrier();
    }
    __syncthreads();                                   // every wavefront is done with the stages
    if constexpr (KG == 2) {
        // group 1 hands its sums over through its stages: piece c of thread t at [c][t]
        int4 *const ex = reinterpret_cast<int4 *>(lds + kStages * kStageT) + tid;
        static_assert(NI * 8 * kThreads * 16 <= kStages * kStageT, "the sums of a group fit its stages");
        if (grp == 1) {
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        ex[((i * 2 + j) * 4 + q) * kThreads] =
                            make_int4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
        }
        __syncthreads();
        if (grp == 1) return;
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int4 v = ex[((i * 2 + j) * 4 + q) * kThreads];
                    acc[i][j][4 * q] += v.x;
                    acc[i][j][4 * q + 1] += v.y;
                    acc[i][j][4 * q + 2] += v.z;
                    acc[i][j][4 * q + 3] += v.w;
                }
    }

    if (SPLIT) {
        // accumulator piece c = (i * 2 + j) * 4 + q of thread t at [c][t]: 16 bytes per lane, contiguous
        int4 *const mine = reinterpret_cast<int4 *>(a.part) + ((int64_t)tile_id * a.splits + split) * (16 * kThreads) + tid;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            if (m0 + wm * (NI * 32) + i * 32 >= a.M) continue;   // no token in these 32 rows: nobody reads them (uniform)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    mine[((i * 2 + j) * 4 + q) * kThreads] =
                        make_int4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
        }
        return;
    }

    // Fused epilogue.  Dequantize with 2^e * sw[n] / 16 in registers (16: the widened weights), then transpose through LDS: a lane holds four
    // consecutive channels of one token (8 bytes), the store wants eight lanes
    // per 128-byte row.  Each wavefront uses a private 64 x 144-byte region.
    const int mrow = m0 + wm * (NI * 32) + (lane & 31);
    if (a.corr) {
        // unsigned activation grid: add corr * sum_k w[n,k], times the 16 the
        // accumulators still carry (|16 acc| <= 16 * 255 * 8 * K < 2^31 for K <= 65536)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int4 ws = *reinterpret_cast<const int4 *>(pwsum + ncol + j * 32 + q * 8);   // padded to 256 channels
                const int t[4] = {ws.x, ws.y, ws.z, ws.w};
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int add = (a.corr * t[r]) << AGQ_W_SHIFT;
#pragma unroll
                    for (int i = 0; i < NI; ++i) acc[i][j][4 * q + r] += add;
                }
            }
    }
    if (pacc) {   // exact accumulators for parity checks (plain stores)
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int m = mrow + i * 32, n = ncol + j * 32 + (r >> 2) * 8 + (r & 3);
                    if (m < a.M && n < pN) pacc[(int64_t)m * pN + n] = acc[i][j][r] >> AGQ_W_SHIFT;
                }
    }
    const float scale16 = a.scale_e * (1.0f / (1 << AGQ_W_SHIFT));   // the factor 16 goes with the scale: exact
    unsigned char *obuf = lds + wave * (NI * 32 * kOutStride);   // 4.5 NI KiB per wavefront
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float g[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const uint32_t pair = r < 2 ? swp[j][q].x : swp[j][q].y;
                    g[r] = scale16 * __half2float(__ushort_as_half((unsigned short)((r & 1) ? pair >> 16 : pair & 0xFFFF)));
                }
                uint2 pk;
                pk.x = agq_dequant2((float)acc[i][j][4 * q], g[0], (float)acc[i][j][4 * q + 1], g[1]);
                pk.y = agq_dequant2((float)acc[i][j][4 * q + 2], g[2], (float)acc[i][j][4 * q + 3], g[3]);
                const int row = i * 32 + (lane & 31), col = j * 32 + q * 8 + (lane >> 5) * 4;
                *reinterpret_cast<uint2 *>(obuf + row * kOutStride + col * 2) = pk;
            }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (pldy & 7) {
        // Rows that do not start on 16 bytes: 32 lanes a row, four bytes a lane and two rows an instruction, from the row's
        // first word boundary on; a row that starts inside a word has single values at both ends.  (2000 tokens,
        // 4096 -> 4100, pre-pass included: 57 us; with eight channels a lane and two bytes a store 69 us; 4096 -> 4096: 40 us.)
        const int nw = n0 + wn * 64, half = lane >> 5;
#pragma unroll 4
        for (int it = 0; it < NI * 16; ++it) {
            const int row = it * 2 + half, m = m0 + wm * (NI * 32) + row;
            if (m >= a.M) break;
            const int odd = (int)((int64_t)m * pldy) & 1;
            const int c0 = 2 * (lane & 31) + odd, c1 = c0 + 1 < 64 ? c0 + 1 : 0;       // the last lane of an odd row: both ends
            const uint16_t *const op = reinterpret_cast<const uint16_t *>(obuf + row * kOutStride);
            const uint32_t v0 = op[c0], v1 = op[c1];
            __half *const yp = py + (int64_t)m * pldy + nw;
            if (c1 && nw + c1 < pN) {
                *reinterpret_cast<uint32_t *>(yp + c0) = v0 | (v1 << 16);
            } else {
                if (nw + c0 < pN) yp[c0] = __ushort_as_half((unsigned short)v0);
                if (c1 == 0 && nw < pN) yp[0] = __ushort_as_half((unsigned short)v1);
            }
        }
        return;
    }
    const int nbase = n0 + wn * 64 + (lane & 7) * 8;          // eight channels per lane
    const bool vec_ok = nbase + 7 < pN;
#pragma unroll
    for (int it = 0; it < NI * 4; ++it) {
        const int row = it * 8 + (lane >> 3);
        const int m = m0 + wm * (NI * 32) + row;
        if (m >= a.M || nbase >= pN) continue;
        const uint4 v = *reinterpret_cast<const uint4 *>(obuf + row * kOutStride + (lane & 7) * 16);
        __half *yp = py + (int64_t)m * pldy + nbase;
        if (vec_ok) {
            *reinterpret_cast<uint4 *>(yp) = v;
        } else {
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
            for (int c = 0; c < 8 && nbase + c < pN; ++c)
                yp[c] = __ushort_as_half((unsigned short)(w[c >> 1] >> (16 * (c & 1))));
        }
    }
}

// Second kernel of a K split: workgroup (tile, piece c) adds the `splits` partial copies of accumulator piece c of
// every thread of the tile's workgroups (same thread numbering, same tile walk as above) and runs the same
// epilogue arithmetic on the sums; a thread owns four consecutive channels of one token.
__global__ __launch_bounds__(kThreads) void split_reduce_kernel(const TiledArgs a) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int tile_id = blockIdx.x >> 4, c = blockIdx.x & 15;
    const int i = c >> 3, j = (c >> 2) & 1, q = c & 3;
    int bid = tile_id;
    // The projection by selects: its fields come with the one round of scalar loads that reads the argument record, where
    // a lookup at an index is a second, dependent one (70 split calls of 40 to 256 rows, 12 to 37 us each: 0.17 us less on
    // average, 8192 -> 1024 at 64 rows 13.10 -> 12.81).  (The tiled kernel above spills with selects and looks up.)
    const int pj = (bid >= a.proj[1].start) + (bid >= a.proj[2].start) + (bid >= a.proj[3].start);
    auto pick = [pj](auto v0, auto v1, auto v2, auto v3) { return pj == 0 ? v0 : (pj == 1 ? v1 : (pj == 2 ? v2 : v3)); };
#define AGQ_PICK(FIELD) pick(a.proj[0].FIELD, a.proj[1].FIELD, a.proj[2].FIELD, a.proj[3].FIELD)
    bid -= AGQ_PICK(start);
    const int pN = AGQ_PICK(N), ptiles_n = AGQ_PICK(tiles_n);
    const uint16_t *const psw = reinterpret_cast<const uint16_t *>(AGQ_PICK(sw));
    __half *const py = AGQ_PICK(y);
    const int64_t pldy = AGQ_PICK(ldy);
    int32_t *const pacc = AGQ_PICK(acc);
    const int32_t *const pwsum = AGQ_PICK(wsum);
#undef AGQ_PICK
    const int band = bid / (kBand * ptiles_n);
    const int rows = min(kBand, a.tiles_m - band * kBand);
    const int within = bid - band * kBand * ptiles_n;
    const int tn = within / rows, tm = band * kBand + within - tn * rows;
    const int m = tm * BM + wm * 64 + i * 32 + (lane & 31);
    const int n = tn * BN + wn * 64 + j * 32 + q * 8 + (lane >> 5) * 4;

    if (m >= a.M || n >= pN) return;
    const int4 *src = reinterpret_cast<const int4 *>(a.part) + ((int64_t)tile_id * a.splits * 16 + c) * kThreads + threadIdx.x;
    int sum[4] = {0, 0, 0, 0};
#pragma unroll 4
    for (int s = 0; s < a.splits; ++s) {
        const int4 v = src[(int64_t)s * (16 * kThreads)];
        sum[0] += v.x;
        sum[1] += v.y;
        sum[2] += v.z;
        sum[3] += v.w;
    }
    uint32_t h[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int nn = min(n + r, pN - 1);   // channels past N are not stored
        if (a.corr) sum[r] += (a.corr * pwsum[nn]) << AGQ_W_SHIFT;
        const int v = sum[r] >> AGQ_W_SHIFT;
        if (pacc && n + r < pN) pacc[(int64_t)m * pN + n + r] = v;
        h[r] = __half_as_ushort(agq_dequant(v, a.scale_e * __half2float(__ushort_as_half((unsigned short)psw[nn]))));
    }
    __half *yp = py + (int64_t)m * pldy + n;
    if ((pldy & 3) == 0 && n + 3 < pN) {
        *reinterpret_cast<uint2 *>(yp) = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
    } else {
        for (int r = 0; r < 4 && n + r < pN; ++r) yp[r] = __ushort_as_half((unsigned short)h[r]);
    }
}

}  // namespace

int agq_launch_gemm_tiled(const void *x_tiles, int64_t M, int64_t K, int e, int corr, const struct agq_proj *projs, int count,
                          int n_extra, AgqTiledVariant variant, const AgqSplitPlan &plan, void *split_ws, void *stream) {
    TiledArgs a = {};
    a.xt = (const agq_u4 *)x_tiles;
    a.M = (int)M;
    a.K = (int)K;
    a.KT = (int)agq_k_tiles(K);
    a.tiles_m = (int)((M + BM - 1) / BM);
    if (variant == TILED_64 || variant == TILED_64X2) a.tiles_m = (int)((M + 63) / 64);
    a.scale_e = ldexpf(1.0f, e);
    a.corr = corr;
    a.n_extra = 0;
    a.trip_shift = nullptr;
    int tiles = 0;
    for (int p = 0; p < kMaxProj; ++p) {
        const agq_proj &pr = projs[p < count ? p : count - 1];
        TiledProj &t = a.proj[p];
        t.start = tiles;
        t.N = (int)pr.N;
        t.tiles_n = (int)((pr.N + BN - 1) / BN);
        if (p < count) tiles += a.tiles_m * t.tiles_n;
        t.blob = (const agq_u4 *)pr.w_packed;
        t.sw = (const __half *)pr.w_scale_f16;
        t.y = (__half *)pr.y_f16;
        t.ldy = pr.ldy;
        t.acc = pr.acc_out;
        t.wsum = n_extra >= 0 ? (const int32_t *)((const char *)pr.w_packed + agq_trip_layout(pr.N, K, n_extra).wsum_off)
                              : agq_blob_wsum(pr.w_packed, pr.N, K);
    }
    const unsigned grid = (unsigned)tiles;
    hipStream_t st = (hipStream_t)stream;
    if (n_extra >= 0) {
        // every blob of the call was packed with the same factors: the shift table of the first serves all
        const AgqTripLayout L = agq_trip_layout(projs[0].N, K, n_extra);
        a.KT = (int)L.KTall;
        a.n_extra = n_extra;
        a.trip_shift = (const int32_t *)((const char *)projs[0].w_packed + L.meta_off) + 16;
    }
    const bool trip = n_extra >= 0;
    if (variant == TILED_SPLIT) {
        a.splits = plan.splits;                          // TRIP: the extra steps and their shifts stay in the first slice
        a.steps_per_split = plan.steps;
        a.tiles_all = tiles;
        a.part = (int32_t *)split_ws;
        if (trip) gemm_tiled_kernel<true, true, 2, 1><<<grid * (unsigned)plan.splits, kThreads, 0, st>>>(a);
        else gemm_tiled_kernel<false, true, 2, 1><<<grid * (unsigned)plan.splits, kThreads, 0, st>>>(a);
        split_reduce_kernel<<<grid * 16, kThreads, 0, st>>>(a);
    } else if (variant == TILED_64X2) {
        if (trip) gemm_tiled_kernel<true, false, 1, 2><<<grid, 2 * kThreads, 0, st>>>(a);
        else gemm_tiled_kernel<false, false, 1, 2><<<grid, 2 * kThreads, 0, st>>>(a);
    } else if (variant == TILED_64) {
        if (trip) gemm_tiled_kernel<true, false, 1, 1><<<grid, kThreads, 0, st>>>(a);
        else gemm_tiled_kernel<false, false, 1, 1><<<grid, kThreads, 0, st>>>(a);
    } else {
        if (trip) gemm_tiled_kernel<true, false, 2, 1><<<grid, kThreads, 0, st>>>(a);
        else gemm_tiled_kernel<false, false, 2, 1><<<grid, kThreads, 0, st>>>(a);
    }
    return (int)hipGetLastError();
}

