// int8-MFMA kernel of the quantized linear layer for many tokens (prompts; bound by the matrix cores, and below a few
// hundred tokens by the time a launch takes to get going).
//
// A workgroup is four wavefronts side by side over the output channels (times KG groups that share K).  A wavefront
// owns 16 NT tokens x 16 JT channels as NT x JT MFMA tiles of 16 x 16 (v_mfma_i32_16x16x64_i8), so a workgroup tile is
// 16 NT tokens x 64 JT channels, K step 128.
//
//   weights go straight from memory into the registers of the one wavefront that multiplies them: lane l's 16 bytes of
//     a chunk of the blob (agq_quant.hip) are channel l & 15, k 16 (l >> 4) .. + 15 of the first 64 (low nibbles) and of
//     the second 64 (high nibbles) of the step, which is what the MFMA takes, P steps ahead.  They are widened to int8
//     in registers (three bit operations per eight weights) once per wavefront, for all of its tokens.
//   activation codes: int8, laid out by the pre-pass in 1 KiB pieces (32 tokens x 32 k; agq_quant.hip), copied to LDS by
//     direct global-to-LDS loads into a ring of Q stages, read by all wavefronts of the group.  Lane l of a fragment
//     (16 tokens x 64 k) reads token l & 15, k 16 (l >> 4): four runs of 256 bytes, every run over all banks, so the
//     sixteen lanes that an LDS cycle serves meet every bank once as they would in one run of 1 KiB.
//
// Why this shape.  With all CUs multiplying the chip runs at its power limit, so what counts is energy per product.  Nothing but
// 16 x 16 x 64 MFMAs on the codes and weights of a layer runs at 2.1 to 2.2 GHz, 4.4-4.6 POP/s, nothing but 32 x 32 x 32 ones at
// 3.7-4.1 (accumulators are read and written once per 64 k instead of per 32; 4.9 both on zeros); this kernel's loop at 1.6 to 1.9 GHz.  A wavefront that
// owns all tokens of the tile needs no weight twice, so weights skip LDS, are widened half as often (128 tokens) as by
// wavefronts of 64 x 64, and a CU loads and reads from LDS a third less.  Against 128 x 128 tiles in 64 x 64 wavefronts with
// both operands through LDS: 2048 x 11008 -> 4096 74 -> 64 us, 4096 -> 12288 89 -> 74, 4096 -> 22016 155 -> 140;
// 1024 x 13824 -> 5120 79 -> 57 (128 x 192 tiles: 216 workgroups instead of 320 on 256 CUs); 300 x 4096 -> 22016 39 -> 32.
#include "../../include/agq.h"
#include "agq_device.h"
#include "agq_internal.h"

#include <utility>

typedef unsigned int agq_u4 __attribute__((ext_vector_type(4)));
typedef unsigned int agq_u4_at_2 __attribute__((ext_vector_type(4), aligned(2)));   // sixteen bytes at any fp16 value

namespace {

constexpr int kThreads = 256;

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
    int M, KT;
    int tiles_m, band;      // token tiles, and how many of them the tile walk takes together
    int whole;              // tiles from here on are dealt out as halves (a multiple of 8)
    int turn;               // two groups: K steps by which a token tile starts further on than the one before it
    float scale_e;
    int corr;               // unsigned activation grid: acc += corr * wsum[n]; 0 on the signed grid
    // TRIP blob: the first n_extra steps are the extra chunks of the channels with a factor;
    // trip_shift[kt] (device) is the left shift of the running accumulators after step kt
    int n_extra;
    const int32_t *trip_shift;
    // K split over `splits` workgroups per tile (few tiles, long K), steps_per_split K steps each: they
    // leave int32 partial tiles in `part`, which a second kernel adds up and dequantizes
    int splits, steps_per_split, tiles_all;
    int32_t *part;       // [tile][split][NT JT][256 threads][4]
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

// vmcnt(n) lgkmcnt(l): bits 3:0 and 15:14 = vmcnt, 6:4 = 7 (no wait), 11:8 = lgkmcnt
constexpr int wait_for(int vm, int lgkm) { return (vm & 15) | ((vm >> 4) << 14) | 0x70 | (lgkm << 8); }

template <int N>
struct Int {
    static constexpr int value = N;
};
template <int N, class F, int... I>
__device__ __forceinline__ void unroll_(F &&f, std::integer_sequence<int, I...>) {
    (f(Int<I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void unroll(F &&f) {
    unroll_<N>(f, std::make_integer_sequence<int, N>{});
}

// Copies of 1 KiB from global memory into LDS in two parts, so that each can hide behind a matrix instruction of its own.
__device__ __forceinline__ uint32_t lds_dma_base(uint32_t lds_addr) {
    uint32_t m0;
    asm volatile("s_mov_b32 m0, %1" : "={m0}"(m0) : "s"(lds_addr));
    return m0;
}
template <int G>
__device__ __forceinline__ void lds_dma16_at(uint32_t m0, uint32_t voff, const void *sbase) {
    asm volatile("global_load_lds_dwordx4 %0, %1 offset:%3" : : "v"(voff), "s"(sbase), "{m0}"(m0), "n"(G) : "memory");
}

// Steps that the weights of a wavefront are requested ahead (it holds P + 1 sets of them), stages of activation codes in
// LDS, and activation fragments in registers (a ring; a power of two that divides the 2 NT of a step).
constexpr int weights_ahead(int NT, int JT, int KG) {
    if (KG == 2) return NT == 2 ? (JT == 1 ? 8 : 6) : 4;
    if (NT == 8) return JT == 4 ? 3 : (JT == 3 ? 4 : 6);
    return JT == 4 ? 4 : (JT == 3 ? 5 : (NT == 2 && JT == 1 ? 10 : 6));
}
constexpr int code_stages(int NT, int KG) { return NT == 8 || (NT == 4 && KG == 2) ? 4 : (NT == 4 ? 6 : 8); }
constexpr int fragment_ring(int NT, int JT) { return NT == 8 && JT == 4 ? 4 : (NT * JT >= 16 ? NT : 2 * NT); }

// TRIP: the blob and the activation stages carry extra steps in front, ordered by
// descending factor; after the last step of a factor the accumulators are shifted
// left by the difference to the next factor (Horner), so that at the end every
// extra step has been multiplied by 2^factor (Section 4.4) - exact in int32.
//
// SPLIT: with few tiles and a long K, a tile's K steps are shared out over several workgroups.  Each stores its int32
// accumulators as a partial tile and is done; split_reduce_kernel, launched behind it, adds the partial tiles up and runs the
// epilogue.  (One kernel in which the last workgroup to arrive at a tile adds the others' partial tiles was measured slower
// than no split at all: it has to read them in dependent rounds through device-scope loads, or with cache-wide write-backs and
// invalidations around them.)  An int32 sum does not depend on its order, so the result is the unsplit kernel's bit for bit.
//
// KG: groups of four wavefronts that share the K steps of the workgroup's tile, each with stages of its own; they meet at the
// same barriers, and at the end each hands the other the sums of half of the token tiles.
//
// The schedule.  A wavefront issues one instruction in about 4.5 cycles and an MFMA waits at issue for the one before it, 16
// cycles: what follows an MFMA is hidden by it up to two or three instructions, and a bunch anywhere leaves the matrix core
// idle.  So the other work of a step is dealt out one MFMA at a time (sched_barrier(0) around each): a fragment read per group
// of JT, the masks of the high nibbles and the weight requests in the first half of the step, shift and mask of the next step's low
// nibbles and the copies in the second.  166 -> 161 instructions a step of 128 x 256 and none of them in bunches: 1208 -> 1146
// cycles, of which 1024 are MFMAs; the meeting costs 30 to 60 of the rest.
//   Loads return in order.  The compiler counts the weight loads and places their waits itself; it does not see the copies,
// so its waits are longer than needed by as many copies as are in between, which is why P is what it is (two instead of three
// steps ahead: 65 -> 67 us on 11008 -> 4096).  The copies are waited for where the wavefronts meet, once a step, by the
// counts below: in front of group B every wavefront has read all of this step's stage, which the copies of the step Q ahead
// then fill, and the codes of the step two ahead have arrived.  The last steps (at most P of them) are code of their own that
// requests no weights: the compiler would drop those loads, which nobody reads, and with them the counts would be wrong.
// GJT: the grid's column tiles are 64 GJT channels wide, and this workgroup takes the half `part_n` of tile `bid` where JT is
// half of GJT, else all of it (part_n 0).
template <bool TRIP, bool SPLIT, int NT, int JT, int KG, int GJT>
__device__ __forceinline__ void tiled_tile(const TiledArgs &a, unsigned char *const lds, int bid, int part_n) {
    constexpr int P = weights_ahead(NT, JT, KG) - (TRIP && NT == 8);   // (the shifts take registers)
    constexpr int SETS = P + 1;                          // register sets of weights
    constexpr int Q = code_stages(NT, KG), R = fragment_ring(NT, JT);
    constexpr int B = 2 * NT - R / 2;                    // group of MFMAs in front of which the wavefronts meet
    constexpr int NC = NT / 2;                           // activation copies of a wavefront per step
    constexpr int BMT = NT * 16, BNT = GJT * 64;
    constexpr int kStageT = NT * 2048;
    constexpr int kRow = JT * 32 + 16;                   // bytes per row of a wavefront's output in LDS
    constexpr int kPass = NT / KG < 4 ? NT / KG : 4;     // 16-token tiles per pass of the epilogue
    constexpr int kGroupLds = Q * kStageT;
    static_assert(SETS >= 3 && P >= Q - 2 && Q >= 3, "the counts of the waits below");
    static_assert(kGroupLds >= 4 * kPass * 16 * kRow, "the epilogue's rows fit the stages");
    static_assert(KG == 1 || NT * JT * 4 * kThreads * 4 <= KG * kGroupLds, "the sums that change hands fit");
    const int lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) & 3);
    const int grp = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    const int tid = threadIdx.x & (kThreads - 1);

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
    const int band = bid / (a.band * ptiles_n);
    const int rows = min(a.band, a.tiles_m - band * a.band);
    const int within = bid - band * a.band * ptiles_n;
    const int tn = within / rows, tm = band * a.band + within - tn * rows;
    const int m0 = tm * BMT, n0 = tn * BNT + part_n * (JT * 64) + (int)wave * (JT * 16);      // channels of this wavefront
    const int KTfull = a.KT;
    const int kwg = SPLIT ? split * a.steps_per_split : 0;
    const int KTwg = SPLIT ? min(a.steps_per_split, KTfull - kwg) : KTfull;  // steps of this workgroup
    // KG == 2: the first half for group 0 (the extra steps, whose shifts apply to what came before them, stay together),
    // the rest for group 1.  (Two steps at least, and the extra steps are never all of them: neither group is empty.)
    const int khalf = KG == 1 ? KTwg : max((KTwg + 1) >> 1, TRIP ? a.n_extra : 0);
    const int kbeg = kwg + (grp == 1 ? khalf : 0);
    const int KT = grp == 1 ? KTwg - khalf : khalf;      // steps of this group

    // Activation: the token tiles of the workgroup are 2 NT KiB in a row of every 16 KiB stage of the pre-pass, a quarter of
    // them per wavefront.  (The pre-pass pads the tokens to 128.)
    const uint32_t voff = (uint32_t)lane * 16;
    const char *const ap = reinterpret_cast<const char *>(a.xt) + ((int64_t)(m0 >> 7) * KTfull + kbeg) * 16384 + (m0 & 127) * 128 + wave * (NC * 1024);
    const __attribute__((address_space(1))) char *bp[JT];
    const int nt_last = ((pN + 255) >> 8) * 16 - 1;      // channel tiles of the blob
#pragma unroll
    for (int j = 0; j < JT; ++j)
        bp[j] = (const __attribute__((address_space(1))) char *)pblob + ((int64_t)min(n0 / 16 + j, nt_last) * KTfull + kbeg) * 1024;
    uint32_t wvoff = voff;
    const uint32_t lds_base = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) unsigned char *)lds) + grp * kGroupLds + wave * (NC * 1024);

    agq_u4 w[SETS][JT];
    agq_v4i xa[R];
    agq_v4i wb[JT];                                      // low nibbles of this step, widened (the high ones in place, in w)
    agq_v4i acc[NT][JT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < JT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][r] = 0;

    auto load_w = [&](agq_u4 (&d)[JT], int j) { d[j] = *(const __attribute__((address_space(1))) agq_u4 *)(bp[j] + wvoff); };
    // Requests past the end repeat the last step.  Two groups: a token tile takes its steps from the `turn`-th of the one
    // before it on (see the launcher); request `jump` is then the last step of K, the one behind it the first.
    const int last = KT - 1;
    constexpr bool TURN = KG == 2 && !TRIP;
    const int first_step = TURN ? a.turn * tm : 0, jump = first_step > 0 ? last - first_step : -1;
    wvoff += first_step * 1024;
    uint32_t avoff = voff + first_step * 16384;
    auto ahead = [&](int k) { return TURN && k == jump ? -last : (k < last ? 1 : 0); };      // from request k to the next, in steps
    auto next_w = [&](int k) { wvoff += ahead(k) * 1024; };
    auto next_a = [&](int k) { avoff += ahead(k) * 16384; };
    auto copy_stage = [&](uint32_t st) {
        unroll<NC>([&](auto p_tag) {
            constexpr int p = decltype(p_tag)::value;
            const uint32_t at = lds_dma_base(lds_base + st);
            asm volatile("s_nop 0");
            lds_dma16_at<p * 1024>(at, avoff, ap);
        });
    };
    constexpr int V = P > Q ? P : Q;
    unroll<V>([&](auto v_tag) {                          // what steps -V .. -1 would have requested
        constexpr int v = decltype(v_tag)::value - V;
        if constexpr (v + P >= 0) {
#pragma unroll
            for (int j = 0; j < JT; ++j) load_w(w[v + P], j);
            next_w(v + P);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (v + Q >= 0) {
            copy_stage((v + Q) * kStageT);
            next_a(v + Q);
        }
        __builtin_amdgcn_sched_barrier(0);
    });
    __builtin_amdgcn_s_waitcnt(wait_for((Q - 2) * (JT + NC), 0));        // stages 0 and 1 are here
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    uint32_t rd = 0;                                     // stage of this step
    const unsigned char *const lrd = lds + grp * kGroupLds + (lane >> 5) * 1024 + ((lane >> 4) & 1) * 512 + (lane & 15) * 16;
    auto frag = [&](const unsigned char *s, int g) {     // group g: half g / NT of the step, 16-token tile g % NT
        const int i = g % NT;
        return *reinterpret_cast<const agq_v4i *>(s + (i >> 1) * 4096 + g / NT * 2048 + (i & 1) * 256);
    };
#pragma unroll
    for (int g = 0; g < R - 1; ++g) xa[g] = frag(lrd, g);
#pragma unroll
    for (int d = 0; d < 4 * JT; ++d) wb[d >> 2][d & 3] = (int)((w[0][d >> 2][d & 3] << 4) & 0xF0F0F0F0u);
    int kt = 0;
    auto step = [&](auto set_tag, auto tail_tag) {
        constexpr bool TAIL = decltype(tail_tag)::value != 0;
        constexpr bool COPY = !TAIL || Q < P;            // at most P steps are left at the tail's start
        constexpr int S = decltype(set_tag)::value, SN = (S + 1) % SETS, SL = (S + P) % SETS;
        constexpr int SLOTS = NT * JT;
        const uint32_t rn = rd == (Q - 1) * kStageT ? 0 : rd + kStageT;
        const unsigned char *const sc = lrd + rd, *const sn = lrd + rn;
        uint32_t part[JT * 4], m0r = 0;
        unroll<2 * SLOTS>([&](auto sl_tag) {
            constexpr int sa = decltype(sl_tag)::value, u = sa / SLOTS, sl = sa % SLOTS, i = sl / JT, j = sl % JT, g = u * NT + i;
            if constexpr (g == B && j == 0) {
                asm volatile("" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
                // newer than the codes of the step two ahead; the tail requests no weights, and those from before it are not counted on
                constexpr int vm = !TAIL ? (Q - 3) * (JT + NC) + JT : (COPY ? (Q - 3) * NC : (Q - 3 > S ? (Q - 3 - S) * NC : 0)), lg = R / 2 - 1;
                __builtin_amdgcn_s_waitcnt(wait_for(vm, lg));
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (j == 0 && (g & 1) == 0) {
                __builtin_amdgcn_s_waitcnt(wait_for(63, R - 3));      // fragments g and g + 1 are here
                __builtin_amdgcn_sched_barrier(0);
            }
            acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(u == 0 ? wb[j] : __builtin_bit_cast(agq_v4i, w[S][j]), xa[g % R], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            // the fragment of the group before this one makes room for the one R - 1 groups ahead
            if constexpr (j == 0) xa[(g + R - 1) % R] = g - 1 + R < 2 * NT ? frag(sc, g - 1 + R) : frag(sn, g - 1 + R - 2 * NT);
            if constexpr (u == 0) {
                // 4 JT words of the high nibbles over SLOTS slots; the weights of the step P ahead
                constexpr int d0 = sl * 4 * JT / SLOTS, d1 = (sl + 1) * 4 * JT / SLOTS;
#pragma unroll
                for (int d = d0; d < d1; ++d) w[S][d >> 2][d & 3] &= 0xF0F0F0F0u;
                constexpr int at = JT > 2 ? 2 : (JT > 1 ? 1 : 0);
                if constexpr (!TAIL && (JT <= NT ? (j == at && i < JT) : (j >= at && (j - at) < 2 && i * 2 + j - at < JT))) load_w(w[SL], JT <= NT ? i : i * 2 + j - at);
                if constexpr (!TAIL && sl == SLOTS - 1) next_w(kt + P);
            } else {
                // 8 JT operations on the low nibbles of the next step: shift, then mask
                constexpr int d0 = sl * 8 * JT / SLOTS, d1 = (sl + 1) * 8 * JT / SLOTS;
#pragma unroll
                for (int o = d0; o < d1; ++o) {
                    const int d = o >> 1;
                    if ((o & 1) == 0) part[d] = w[SN][d >> 2][d & 3] << 4;
                    else wb[d >> 2][d & 3] = (int)(part[d] & 0xF0F0F0F0u);
                }
                // the copies of the step Q ahead into the stage that everybody has read: one a slot
                constexpr int first = (B - NT) * JT, n = SLOTS - first, by = n / (NC + 1) > 0 ? n / (NC + 1) : 1;
                static_assert(n >= NC + 1 || n >= 2, "room for the copies");
                if constexpr (COPY && sl == first) m0r = lds_dma_base(lds_base + rd);
                if constexpr (COPY && n >= NC + 1) {
                    if constexpr (sl > first && (sl - first) % by == 0 && (sl - first) / by <= NC) lds_dma16_at<((sl - first) / by - 1) * 1024>(m0r, avoff, ap);
                } else if constexpr (COPY && sl == SLOTS - 1) {
                    unroll<NC>([&](auto p_tag) { lds_dma16_at<decltype(p_tag)::value * 1024>(m0r, avoff, ap); });
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (TRIP) {
            if (split == 0 && grp == 0 && kt < a.n_extra) {
                const int sh = a.trip_shift[kt];
                if (sh) {
#pragma unroll
                    for (int i = 0; i < NT; ++i)
#pragma unroll
                        for (int j = 0; j < JT; ++j)
#pragma unroll
                            for (int r = 0; r < 4; ++r) acc[i][j][r] <<= sh;
                }
            }
        }
        // (a value that only the next step uses would move there, behind the loop's branch, with its wait)
#pragma unroll
        for (int j = 0; j < JT; ++j) asm volatile("" : "+v"(wb[j]));
        if constexpr (COPY) next_a(kt + Q);
        rd = rn;
        ++kt;
    };
    // (left in the middle instead of these two loops, the steps' waits became those of the worst path: 65 -> 73 us)
    while (kt + SETS <= KT) unroll<SETS>([&](auto s_tag) { step(s_tag, Int<0>{}); });
    unroll<SETS - 1>([&](auto s_tag) {
        if (kt < KT) step(s_tag, Int<1>{});
    });
    if constexpr (KG == 2) {
        // the groups meet once per step and once before the first one: the shorter one catches up
        for (int more = KTwg - 2 * KT; more > 0; --more) __builtin_amdgcn_s_barrier();
    }
    // per-channel scales of this lane's output columns (accumulator register r of tile j: channel 16 j + 4 (lane >> 4) + r)
    const int ncol = n0 + (lane >> 4) * 4;
    uint2 swp[JT];
#pragma unroll
    for (int j = 0; j < JT; ++j) {
        const int n = ncol + j * 16;
        const uint16_t *sp = reinterpret_cast<const uint16_t *>(psw);
        if ((pN & 3) == 0) {
            swp[j] = *reinterpret_cast<const uint2 *>(sp + min(n, pN - 4));   // 8-byte aligned: n % 4 == 0
        } else {
            uint32_t h[4];
            for (int r = 0; r < 4; ++r) h[r] = sp[min(n + r, pN - 1)];
            swp[j] = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
        }
    }
    __builtin_amdgcn_s_waitcnt(wait_for(0, 0));
    __syncthreads();
    // Two groups: each finishes half of the token tiles, on the sums that the other one hands over through LDS.
    constexpr int FT = NT / KG;                          // token tiles that this wavefront finishes
    agq_v4i fin[FT][JT];
    if constexpr (KG == 1) {
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int j = 0; j < JT; ++j) fin[i][j] = acc[i][j];
    } else {
        agq_v4i *const ex = reinterpret_cast<agq_v4i *>(lds) + tid;
#pragma unroll
        for (int i = 0; i < FT; ++i)
#pragma unroll
            for (int j = 0; j < JT; ++j) {
                ex[((grp * FT + i) * JT + j) * kThreads] = grp ? acc[i][j] : acc[FT + i][j];
                fin[i][j] = grp ? acc[FT + i][j] : acc[i][j];
            }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < FT; ++i)
#pragma unroll
            for (int j = 0; j < JT; ++j) fin[i][j] += ex[(((grp ^ 1) * FT + i) * JT + j) * kThreads];
        __syncthreads();                                 // the output rows go where the sums were
    }
    const int mf = m0 + grp * (FT * 16);                 // first token of theirs
    if constexpr (SPLIT) {
        int4 *const mine = reinterpret_cast<int4 *>(a.part) + ((int64_t)tile_id * a.splits + split) * (NT * JT * kThreads) + tid;
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            if (m0 + i * 16 >= a.M) continue;
#pragma unroll
            for (int j = 0; j < JT; ++j) mine[(i * JT + j) * kThreads] = make_int4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
        }
        return;
    }
    if (n0 >= pN) return;
    if (a.corr) {
        // unsigned activation grid: add corr * sum_k w[n,k], times the 16 the
        // accumulators still carry (|16 acc| <= 16 * 255 * 8 * K < 2^31 for K <= 65536)
#pragma unroll
        for (int j = 0; j < JT; ++j) {
            const int4 ws = *reinterpret_cast<const int4 *>(pwsum + min(ncol + j * 16, (nt_last + 1) * 16 - 4));   // padded to 256 channels
            const int t[4] = {ws.x, ws.y, ws.z, ws.w};
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int add = (a.corr * t[r]) << AGQ_W_SHIFT;
#pragma unroll
                for (int i = 0; i < FT; ++i) fin[i][j][r] += add;
            }
        }
    }
    if (pacc) {   // exact accumulators for parity checks (plain stores)
#pragma unroll
        for (int i = 0; i < FT; ++i)
#pragma unroll
            for (int j = 0; j < JT; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int m = mf + i * 16 + (lane & 15), n = ncol + j * 16 + r;
                    if (m < a.M && n < pN) pacc[(int64_t)m * pN + n] = fin[i][j][r] >> AGQ_W_SHIFT;
                }
    }
    // Fused epilogue.  Dequantize with 2^e * sw[n] / 16 in registers (16: the widened weights), then transpose through LDS: a
    // lane holds four consecutive channels of one token (8 bytes), the store wants 16 bytes a lane.  A wavefront stores its own
    // channels from its own rows; where rows do not start on sixteen bytes the stores still take that much at once (1200 x 1280 ->
    // 4100 with 128 x 192 tiles 13.5 us; a word a lane, aligned, 19.3).
    const float scale16 = a.scale_e * (1.0f / (1 << AGQ_W_SHIFT));
    unsigned char *const obuf = lds + (grp * 4 + wave) * (kPass * 16 * kRow);
#pragma unroll
    for (int i0 = 0; i0 < FT; i0 += kPass) {
        constexpr int nrows = kPass * 16;
#pragma unroll
        for (int ii = 0; ii < kPass; ++ii) {
#pragma unroll
            for (int j = 0; j < JT; ++j) {
                float g[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const uint32_t pair = r < 2 ? swp[j].x : swp[j].y;
                    g[r] = scale16 * __half2float(__ushort_as_half((unsigned short)((r & 1) ? pair >> 16 : pair & 0xFFFF)));
                }
                const agq_v4i &v = fin[i0 + ii][j];
                uint2 pk;
                pk.x = agq_dequant2((float)v[0], g[0], (float)v[1], g[1]);
                pk.y = agq_dequant2((float)v[2], g[2], (float)v[3], g[3]);
                *reinterpret_cast<uint2 *>(obuf + (ii * 16 + (lane & 15)) * kRow + (j * 16 + (lane >> 4) * 4) * 2) = pk;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int mb = mf + i0 * 16;
        constexpr int kPieces = JT * 2;              // eight channels each, per row
#pragma unroll
        for (int it = 0; it * 64 < nrows * kPieces; ++it) {
            const int piece = it * 64 + lane, row = piece / kPieces, nbase = n0 + (piece - row * kPieces) * 8, m = mb + row;
            if (row >= nrows || m >= a.M || nbase >= pN) continue;
            const uint4 v = *reinterpret_cast<const uint4 *>(obuf + row * kRow + (piece - row * kPieces) * 16);
            __half *yp = py + (int64_t)m * pldy + nbase;
            if (nbase + 7 < pN) {
                *reinterpret_cast<agq_u4_at_2 *>(yp) = agq_u4_at_2{v.x, v.y, v.z, v.w};
            } else {
                const uint32_t u[4] = {v.x, v.y, v.z, v.w};
                for (int c = 0; c < 8 && nbase + c < pN; ++c)
                    yp[c] = __ushort_as_half((unsigned short)(u[c >> 1] >> (16 * (c & 1))));
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}


// HALVES: the tiles from a.whole on, a last round that fills at most half of the CUs, are dealt out as halves (half of the
// channels each) to twice as many workgroups; see agq_tiled_halves.
template <bool TRIP, bool SPLIT, int NT, int JT, int KG, bool HALVES>
__global__ __launch_bounds__(kThreads * KG, 2) void gemm_tiled_kernel(const TiledArgs a) {
    __shared__ __align__(16) unsigned char lds[KG * code_stages(NT, KG) * NT * 2048];
    // XCD-aware tile order.  Consecutive workgroup ids land on different XCDs (round-robin over 8), each with its own L2, so
    // first give every XCD a contiguous run of logical tile ids (the first nblk % 8 of them one more); then walk the tile grid
    // in bands of token tiles, column by column, so that a run re-reads as little of either operand as possible.
    const int whole = HALVES ? a.whole : (int)gridDim.x;
    const bool half = HALVES && (int)blockIdx.x >= whole;
    const int nblk = half ? (int)gridDim.x - whole : whole;
    int bid = half ? (int)blockIdx.x - whole : (int)blockIdx.x;
    bid = (bid & 7) * (nblk >> 3) + min(bid & 7, nblk & 7) + (bid >> 3);
    if constexpr (HALVES) {
        if (half) {
            tiled_tile<TRIP, SPLIT, NT, JT / 2, KG, JT>(a, lds, whole + (bid >> 1), bid & 1);
            return;
        }
    }
    tiled_tile<TRIP, SPLIT, NT, JT, KG, JT>(a, lds, bid, 0);
}

// Second kernel of a K split: workgroup (tile, piece c) adds the `splits` partial copies of accumulator piece c of
// every thread of the tile's workgroups (same thread numbering, same tile walk as above) and runs the same
// epilogue arithmetic on the sums; a thread owns four consecutive channels of one token.
template <int NT, int JT>
__global__ __launch_bounds__(kThreads) void split_reduce_kernel(const TiledArgs a) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int tile_id = blockIdx.x / (NT * JT), c = blockIdx.x % (NT * JT);
    const int i = c / JT, j = c % JT;
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
    const int band = bid / (a.band * ptiles_n);
    const int rows = min(a.band, a.tiles_m - band * a.band);
    const int within = bid - band * a.band * ptiles_n;
    const int tn = within / rows, tm = band * a.band + within - tn * rows;
    const int m = tm * (NT * 16) + i * 16 + (lane & 15);
    const int n = tn * (JT * 64) + wave * (JT * 16) + j * 16 + (lane >> 4) * 4;

    if (m >= a.M || n >= pN) return;
    const int4 *src = reinterpret_cast<const int4 *>(a.part) + ((int64_t)tile_id * a.splits * (NT * JT) + c) * kThreads + threadIdx.x;
    int sum[4] = {0, 0, 0, 0};
#pragma unroll 4
    for (int s = 0; s < a.splits; ++s) {
        const int4 v = src[(int64_t)s * (NT * JT * kThreads)];
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
                          int n_extra, const AgqTiledChoice &choice, void *split_ws, void *stream) {
    const bool trip = n_extra >= 0, split = choice.variant == TILED_SPLIT;
    const int tile_m = choice.nt * 16, tile_n = choice.jt * 64;
    TiledArgs a = {};
    a.xt = (const agq_u4 *)x_tiles;
    a.M = (int)M;
    a.KT = (int)agq_k_tiles(K);
    a.tiles_m = (int)((M + tile_m - 1) / tile_m);
    int64_t n_sum = 0;
    for (int p = 0; p < count; ++p) n_sum += projs[p].N;
    a.band = agq_tiled_band(M, n_sum, choice.nt, choice.kg);
    a.scale_e = ldexpf(1.0f, e);
    a.corr = corr;
    int tiles = 0;
    for (int p = 0; p < kMaxProj; ++p) {
        const agq_proj &pr = projs[p < count ? p : count - 1];
        TiledProj &t = a.proj[p];
        t.start = tiles;
        t.N = (int)pr.N;
        t.tiles_n = (int)((pr.N + tile_n - 1) / tile_n);
        if (p < count) tiles += a.tiles_m * t.tiles_n;
        t.blob = (const agq_u4 *)pr.w_packed;
        t.sw = (const __half *)pr.w_scale_f16;
        t.y = (__half *)pr.y_f16;
        t.ldy = pr.ldy;
        t.acc = pr.acc_out;
        t.wsum = trip ? (const int32_t *)((const char *)pr.w_packed + agq_trip_layout(pr.N, K, n_extra).wsum_off)
                      : agq_blob_wsum(pr.w_packed, pr.N, K);
    }
    if (trip) {
        // every blob of the call was packed with the same factors: the shift table of the first serves all
        const AgqTripLayout L = agq_trip_layout(projs[0].N, K, n_extra);
        a.KT = (int)L.KTall;
        a.n_extra = n_extra;
        a.trip_shift = (const int32_t *)((const char *)projs[0].w_packed + L.meta_off) + 16;
    }
    if (choice.kg == 2 && !trip && a.tiles_m > 1) {
        // Workgroups that need the same weights (the token tiles of a column) would request them in the same moment, five at a
        // time with a fifth of the weights in flight.  Started apart in K, each brings in what the others read later: as far
        // apart as the steps go round, as long as what is in between (64 bytes per channel, step and group, an eighth of it
        // per XCD) stays in an XCD's L2.  300 x 11008 -> 4096 27.5 -> 22.2 us, 213 tokens 20.6 -> 18.1, 100 tokens 16.2 -> 14.8, 333 x 5120 -> 5120
        // 15.8 -> 14.3, 333 x 13824 -> 5120 33.3 -> 31; level where K is 4096.  (One group gains less, 128-token tiles lose: more than
        // five of them, and L2 does not hold what lies between; 1024 x 13824 -> 5120 56.5 -> 58.2.)
        const int64_t steps = a.KT / 2, apart = a.tiles_m - 1;
        int64_t turn = steps / a.tiles_m;
        if (turn > 2500000 / (16 * n_sum * apart)) turn = 2500000 / (16 * n_sum * apart);
        a.turn = (int)turn;
    }
    unsigned grid = (unsigned)tiles;
    if (split) {
        a.splits = choice.splits;                        // TRIP: the extra steps and their shifts stay in the first slice
        a.steps_per_split = choice.steps;
        a.tiles_all = tiles;
        a.part = (int32_t *)split_ws;
        grid *= (unsigned)choice.splits;
    }
    hipStream_t st = (hipStream_t)stream;
    bool found = false;
    auto launch = [&](auto nt, auto jt, auto kg, auto sp) {
        constexpr int NT = decltype(nt)::value, JT = decltype(jt)::value, KG = decltype(kg)::value;
        constexpr bool SPLIT = decltype(sp)::value != 0;
        if (found || split != SPLIT || choice.nt != NT || choice.jt != JT || choice.kg != KG) return;
        found = true;
        if constexpr (NT == 8 && JT == 4) {
            a.whole = tiles - (int)agq_tiled_halves(tiles);
            if (a.whole < tiles) {
                const unsigned more = grid + (unsigned)(tiles - a.whole);
                if (trip) gemm_tiled_kernel<true, SPLIT, NT, JT, KG, true><<<more, kThreads * KG, 0, st>>>(a);
                else gemm_tiled_kernel<false, SPLIT, NT, JT, KG, true><<<more, kThreads * KG, 0, st>>>(a);
                return;
            }
        }
        if (trip) gemm_tiled_kernel<true, SPLIT, NT, JT, KG, false><<<grid, kThreads * KG, 0, st>>>(a);
        else gemm_tiled_kernel<false, SPLIT, NT, JT, KG, false><<<grid, kThreads * KG, 0, st>>>(a);
    };
#define AGQ_SHAPE(NT, JT, KG) launch(Int<NT>{}, Int<JT>{}, Int<KG>{}, Int<0>{});
    AGQ_TILED_SHAPES(AGQ_SHAPE)
#undef AGQ_SHAPE
    launch(Int<4>{}, Int<2>{}, Int<1>{}, Int<1>{});
    launch(Int<4>{}, Int<1>{}, Int<1>{}, Int<1>{});
    if (!found) return (int)hipErrorInvalidValue;
    if (split && choice.jt == 2) split_reduce_kernel<4, 2><<<(unsigned)tiles * 8, kThreads, 0, st>>>(a);
    else if (split) split_reduce_kernel<4, 1><<<(unsigned)tiles * 4, kThreads, 0, st>>>(a);
    return (int)hipGetLastError();
}
