// Attention from quantized Q and K in one kernel: integer Q K^T on the int8
// matrix cores (Section 4.2 lists QK among the quantized products), softmax in
// floating point (Section 3.3: non-linear operators stay in floating point),
// Eq.3 (Section 4.1) on the probabilities, the product with the int8 value
// matrix, and the importance of every token on the quantized map (Section 4.3).
// The probabilities never exist in memory.
//
//   s[i,j] = sum_d q[i,d] k[j,d]                         (int32, exact)
//   t[i,j] = -log2 softmax_j(s 2^(e_q+e_k) / sqrt(D)) = L[i] - kappa s[i,j],
//            kappa = 2^(e_q+e_k) log2(e) / sqrt(D),  L[i] = log2 sum_j 2^(kappa s[i,j])
//   c[i,j] = CLIP(round(t), 0, qmax),   o[i,:] = 2^(e_v-qmax) sum_j 2^(qmax-c[i,j]) v[j,:]
//
// Two passes over the key tiles of a 128-row block: the first keeps a running
// maximum and sum per row (L), the second recomputes the scores, turns them
// into the weights 2^(qmax-c) and multiplies.  L and t are evaluated in fp32
// (hardware exp2 / log2), so a code can differ from a float64 evaluation where t lies within the evaluation's error of a
// rounding boundary: about 1e-5 where kappa > 1, 1e-5 + 2^-22 max |kappa s| up to there (see WIDE); everything after the
// codes is exact.
//
// Scores are computed transposed, S^T = K Q^T, with the 32x32x32 int8 MFMA: a lane
// then holds, for its query (column l & 31), the keys 8 q + 4 g + r (g = l >> 5,
// register 4 q + r) of a 32-key sub-tile - which is already the layout of the
// first operand of the 32x32x16 fp16 MFMA if its sixteen k slots are dealt to keys
// in that order (slot 8 g + 4 q' + r of step u <-> key 16 u + 8 q' + 4 g + r).  The
// V tile in LDS is written in that slot order, so no shuffle is needed between
// the two products.
//
// What bounds it: the vector ALU and the matrix cores of a SIMD, which two wavefronts of different
// workgroups keep busy in turn.  Measured: a wavefront by itself issues an instruction every 4.5 cycles, and every
// eight where it needs the one before; conversions, permutes and packed fp16 take the ALU 4.4 cycles, plain
// fp32 2.5, the exponential 8.5, an MFMA eight of the ALU's and 33 of the matrix core's.  So the work of a step is
// dealt out one MFMA at a time, the scores of the next sub-tile beside the arithmetic of this one; scores become floats
// by a subtraction; a conversion to bytes rounds and packs the weights' exponents; V is widened by one
// packed multiply-add.  Against a kernel with nothing dealt out and three workgroups on a CU (the same results bit for
// bit): 40 x 2048 x 128 causal 67.2 -> 59.6 us, 40 x 2048 x 64 55 -> 40 (half of the output blocks were empty there),
// 32 x 384 x 128 14.7 -> 12.6, one head of 128 tokens 7.03 -> 6.85 (without causality 6.18 -> 6.30, the one call that is slower);
// with the code map 107 -> 100, 99 -> 92, 19.3 -> 15.6 and 8.50 -> 7.77.  What is left of a large causal call is the chain of its longest row blocks (32 tiles
// take 45 us alone on a CU, 305 instructions a tile in pass 2).  Not kept: a reference score in place of the running maximum, with differences to it straight from
// the accumulators (58 us, and three times fewer codes off, but other codes than before); one block on eight
// wavefronts, the key tiles shared by two groups of four (72 us then: both wavefronts of a SIMD want the same unit at
// the same time); V tiles straight into registers (no difference).
#include "agq_device.h"
#include "agq_internal.h"

AgqQuant agq_make_quant_signed(int bits, int e, int zp);   // agq_quant.hip

#include <math.h>

#include <type_traits>

typedef _Float16 agq_v8h __attribute__((ext_vector_type(8)));
typedef _Float16 agq_v2h __attribute__((ext_vector_type(2)));
typedef float agq_v16f __attribute__((ext_vector_type(16)));
typedef int agq_v16i __attribute__((ext_vector_type(16)));
typedef uint32_t agq_u4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int kQRows = 128;     // query rows per workgroup (32 per wavefront)
constexpr int kKeys = 64;       // keys per tile: two 32-key sub-tiles
constexpr int kRing = 4;        // K tiles in LDS

struct QkArgs {
    const int8_t *q, *k, *v;   // [H,S,D] each
    __half *o;                 // [S, H*D]
    uint8_t *codes;            // [H,S,S/2] or null
    int32_t *score;            // [S] or null (accumulated with atomics: the caller zeroes it)
    int H, S;
    int causal, qmax;
    float kappa;               // 2^(e_q+e_k) log2(e) / sqrt(D)
    float out_scale;           // 2^(e_v - qmax + 9)
    int ncu;
    char *tiles;               // where Eq.2's codes of o go as well, in the operand order of the tiled GEMM, or null
    AgqQuant quant;
};

template <int N>
struct Int {
    static constexpr int value = N;
};

// Between two tiles: at most VM of this wavefront's loads may still fly (they return in order), its LDS reads and writes
// are done; then meet the others.  (Stores of the code map count as well and come behind the copies: with them a tile waits for
// the copy it has just requested, too.)
template <int VM>
__device__ __forceinline__ void meet() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt((VM & 15) | ((VM >> 4) << 14) | 0x70);   // vmcnt(VM) lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// DT = D / 32: int8 MFMA steps per score tile and 32-channel blocks of the output
// CODES: the code map goes out as well; TILES: Eq.2's codes of o (a.tiles).
// WIDE: kappa > 1.  Up to there kappa times the row's maximum M is rounded by itself, once in pass 1 and once in pass 2 with
// the constant it goes into: t is off by up to three roundings of kappa M, about 2^-14 where |kappa s| reaches 2^8, as it does for
// activations, and below 0.4 at most (|s| <= 2^21), so that no exponent passes the largest weight's.  Beyond, those roundings
// have no bound, and the difference to the maximum, exact in fp32, is taken before the product: the same number of
// instructions, and nothing to cut off, as no difference is above 0.
template <int DT, bool CODES, bool TILES, bool WIDE>
__global__ __launch_bounds__(256, 2) void qk_log2_attn_kernel(const QkArgs a) {
    constexpr int D = DT * 32;
    constexpr int kKTile = kKeys * D;                            // bytes of a K tile
    constexpr int kVTile = D * kKeys * 2;                        // bytes of a V tile, fp16 [channel][slot]
    constexpr int kKC = kKTile / 4096;                           // copies of a K tile per wavefront
    __shared__ __align__(16) uint8_t kt[kRing * kKTile];
    __shared__ __align__(16) uint8_t vt[2 * kVTile];
    __shared__ __align__(16) uint8_t vq[2 * kKTile];                // V tiles as they come
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int S = a.S, H = a.H;
    const int nb = S / kQRows;

    // workgroup -> (head, row block); causal blocks ranked by length and dealt so that
    // the workgroups a CU receives together carry equal work (see the other attention kernel)
    int rank = (int)blockIdx.x;
    if (a.causal) {
        const int run = rank / a.ncu, base = run * a.ncu;
        if (run & 1) rank = base + min(a.ncu, (int)gridDim.x - base) - 1 - (rank - base);
    }
    const int h = rank % H;
    const int b = a.causal ? nb - 1 - rank / H : rank / H;
    const int q0 = b * kQRows;
    const int r0 = __builtin_amdgcn_readfirstlane(q0 + wave * 32);
    const int row = r0 + (lane & 31);                            // this lane's query
    const int c = lane & 31, g = lane >> 5;
    const int nt = (a.causal ? q0 + kQRows : S) / kKeys;         // key tiles of the block
    const int n_main = a.causal ? nt - 2 : nt;                   // tiles that are live for every row of the block
    const int last_sub = a.causal ? r0 >> 5 : 2 * nt - 1;        // last sub-tile with a live key for this wavefront

    const int8_t *qh = a.q + (int64_t)h * S * D;
    const int8_t *kh = a.k + (int64_t)h * S * D;
    const int8_t *vh = a.v + (int64_t)h * S * D;

    // Q: second operand of S^T = K Q^T (column = query l & 31, sixteen d of k-group g per step)
    agq_v4i qf[DT];
#pragma unroll
    for (int s = 0; s < DT; ++s) qf[s] = *reinterpret_cast<const agq_v4i *>(qh + (int64_t)row * D + 32 * s + 16 * g);

    // K tiles: copied straight into a ring of four in LDS, for both passes in one sequence (tile T of the sequence is key
    // tile T, or T - nt in pass 2).  Sixteen lanes read LDS at a time, 256 bytes; the sixteen-byte pieces of a key's row
    // are permuted by the key so that a fragment read (one piece of sixteen keys) meets every bank once: piece i of
    // row r lies at i ^ (r >> 1 & 7) where two rows fill the banks (D = 128), at i ^ (r >> 2 & 3) where four do.  A row stays
    // inside its own cache line on the way.
    constexpr int kPieces = D / 16;
    const int kr = lane / kPieces;                               // row among those that a copy holds: eight or sixteen
    uint32_t k_src[kKC];
#pragma unroll
    for (int i = 0; i < kKC; ++i) {
        const int sw = kPieces == 8 ? (4 * i + (kr >> 1)) & 7 : (kr >> 2) & 3;
        k_src[i] = (uint32_t)(kr * D + (((lane & (kPieces - 1)) ^ sw) << 4));
    }
    const uint32_t wave_u = __builtin_amdgcn_readfirstlane((uint32_t)wave);
    const uint32_t k_lds = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint8_t *)kt) + wave_u * (kKC * 1024);
    const uint32_t kv_bytes = (uint32_t)nt * kKTile;             // of the block's keys: at most 4 MiB
    uint32_t k_at = 0, k_slot = 0;
    auto copy_k = [&] {                                          // the next tile of the sequence; past its end into a slot nobody reads
        const int8_t *const src = kh + wave_u * (kKC * 1024) + k_at;
        lds_dma16_s<0, 0>(k_src[0], src, k_lds + k_slot);
        if constexpr (kKC == 2) lds_dma16_s<0, 1024>(k_src[kKC - 1], src, k_lds + k_slot);
        k_at = k_at + kKTile == kv_bytes ? 0 : k_at + kKTile;
        k_slot = (k_slot + kKTile) & (kRing * kKTile - 1);
    };
    uint32_t k_rd[DT];                                           // operand reads: sixteen d of k-group g of step s, key l & 31
    const int swz = kPieces == 8 ? (c >> 1) & 7 : (c >> 2) & 3;
#pragma unroll
    for (int s = 0; s < DT; ++s) k_rd[s] = (uint32_t)(c * D + (((2 * s + g) ^ swz) << 4));
    agq_v4i kf[DT];
    auto read_k = [&](int s, const uint8_t *tile, int sub) { kf[s] = *reinterpret_cast<const agq_v4i *>(tile + k_rd[s] + sub * (32 * D)); };

    // score tile of 32 keys, transposed: register 4 q + r = key 8 q + 4 g + r, this lane's query
    agq_v16i acc0, acc1, acc2, acc3, cinit;
    auto mfma_s = [&](int s, agq_v16i &acc) {
        acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(kf[s], qf[s], s == 0 ? cinit : acc, 0, 0, 0);
    };

    // V tiles: copied as they are into one of two buffers, then int8 [key][d] -> fp16 [d][slot].  A thread's unit is (chunk of
    // eight slots, NB channels); the eight slots of chunk ch = 4 sub + 2 u + g' hold the keys
    // 32 sub + 16 u + 8 (i >> 2) + 4 g' + (i & 3), i = 0..7 (see the header).  Channel NB c + n is column c of output block
    // n, row 32 n + c of the tile; chunk ch of a row lies at place ch ^ (row >> 1 & 7), for the same reason as K's
    // pieces.
    constexpr int NB = DT;
    const uint32_t vq_lds = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint8_t *)vq) + wave_u * (kKC * 1024);
    uint32_t v_at = 0, v_slot = 0;
    auto copy_v = [&] {                                          // the next tile; past the last one nobody reads it
        const int8_t *const src = vh + wave_u * (kKC * 1024) + v_at;
        lds_dma16_s<0, 0>((uint32_t)lane * 16, src, vq_lds + v_slot);
        if constexpr (kKC == 2) lds_dma16_s<0, 1024>((uint32_t)lane * 16, src, vq_lds + v_slot);
        v_at = v_at + kKTile == kv_bytes ? 0 : v_at + kKTile;
        v_slot ^= kKTile;
    };
    const int vu_c = threadIdx.x & 31, vu_ch = threadIdx.x >> 5;
    const uint8_t *const v_src = vq + (32 * (vu_ch >> 2) + 16 * ((vu_ch >> 1) & 1) + 4 * (vu_ch & 1)) * D + NB * vu_c;
    uint8_t *const v_dst = vt + vu_c * 128 + ((vu_ch ^ ((vu_c >> 1) & 7)) << 4);
    uint32_t vx[8];
    auto read_v = [&](int t) {                                   // bytes v + 128
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint8_t *const p = v_src + (t & 1) * kKTile + (8 * (i >> 2) + (i & 3)) * D;
            vx[i] = (NB == 4 ? *reinterpret_cast<const uint32_t *>(p) : *reinterpret_cast<const uint16_t *>(p)) ^ 0x80808080u;
        }
    };
    // as the low byte of a half, v + 128 is the number (v + 128) 2^-24, and one fused multiply-add makes it v 2^-9
    auto store_v = [&](int t, auto bb_tag) {
        constexpr int bb = decltype(bb_tag)::value;
        agq_u4 out;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t w = __builtin_amdgcn_perm(vx[2 * i + 1], vx[2 * i], 0x0C000C00u | (uint32_t)bb | ((uint32_t)(4 + bb) << 16));
            out[i] = __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(__builtin_bit_cast(agq_v2h, w), agq_v2h{(_Float16)32768.0f, (_Float16)32768.0f},
                                                                            agq_v2h{(_Float16)-0.25f, (_Float16)-0.25f}));
        }
        *reinterpret_cast<agq_u4 *>(v_dst + (t & 1) * kVTile + bb * (32 * 128)) = out;
    };

    copy_k();
    copy_k();
    meet<0>();                                                   // K tiles 0 and 1 and Q have landed
    copy_k();
    copy_v();
    copy_v();

    // The accumulators start at the bit pattern of 1.5 * 2^23: read as floats they are 1.5 * 2^23 + s, and a subtraction
    // makes that (float)s for half the time of a conversion.  As integers they order like the scores.
    constexpr int kBias = 0x4B400000;
#pragma unroll
    for (int r = 0; r < 16; ++r) cinit[r] = kBias;
    float kappa = a.kappa;                                       // in a vector register: a product of three of those is the faster one
    asm("" : "+v"(kappa));
    auto scaled = [&](float s, float plus) { return WIDE ? kappa * s : fmaf(kappa, s, plus); };   // WIDE: s is a difference to the maximum

    // ---- pass 1: per row the maximum score M (an integer) and sum_j 2^(kappa (s_j - M))
    constexpr int kMasked = -(1 << 30);                          // stands for -infinity (|s| < 2^23)
    int run_m = kMasked;
    float run_s = 0.f;
    auto tile_scores = [&](const uint8_t *tile, agq_v16i &s0, agq_v16i &s1) {   // both sub-tiles of a tile at once
        agq_v4i k1[DT];
#pragma unroll
        for (int s = 0; s < DT; ++s) {
            read_k(s, tile, 0);
            k1[s] = *reinterpret_cast<const agq_v4i *>(tile + k_rd[s] + 32 * D);
        }
#pragma unroll
        for (int s = 0; s < DT; ++s) {
            mfma_s(s, s0);
            s1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(k1[s], qf[s], s == 0 ? cinit : s1, 0, 0, 0);
        }
    };
    tile_scores(kt, acc0, acc1);
    // A sub-tile at the diagonal; keys past the query do not count.  Alone on its SIMD a wavefront pays for every instruction: one
    // comparison and a select per score, and the difference to the maximum in one subtraction of floats (one head of 128
    // tokens 7.97 -> 7.22 us against integers and a conversion).
    auto stats = [&](const agq_v16i &acc, int sub, bool masked) {
        const int left = masked ? row - (32 * sub + 4 * g) : 32;
        auto dead = [&](int r) { return 8 * (r >> 2) + (r & 3) > left; };
        int mx = run_m + kBias;
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = max(mx, dead(r) ? kMasked + kBias : acc[r]);
        const int nm = mx - kBias;
        const float ref = AGQ_MAGIC + (float)nm;                 // exact where a score counts, and so is the difference
        float add = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float term = __builtin_amdgcn_exp2f(kappa * (__int_as_float(acc[r]) - ref));
            add += dead(r) ? 0.f : term;
        }
        // nothing counted so far (run_m == kMasked) means run_s == 0: the factor does not matter
        run_s = run_s * __builtin_amdgcn_exp2f(kappa * (float)(run_m - nm)) + add;
        run_m = nm;
    };
    auto tile_stats = [&](const agq_v16i &cur0, const agq_v16i &cur1) {   // a whole live tile
        int mx = run_m + kBias;
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = max(mx, max(cur0[r], cur1[r]));
        const int nm = mx - kBias;
        const float ref = WIDE ? AGQ_MAGIC + (float)nm : AGQ_MAGIC, nmf = WIDE ? 0.f : -kappa * (float)nm;
        float add0 = 0.f, add1 = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            add0 += __builtin_amdgcn_exp2f(scaled(__int_as_float(cur0[r]) - ref, nmf));
            add1 += __builtin_amdgcn_exp2f(scaled(__int_as_float(cur1[r]) - ref, nmf));
        }
        run_s = run_s * __builtin_amdgcn_exp2f(kappa * (float)(run_m - nm)) + (add0 + add1);
        run_m = nm;
    };
    // A tile that is live for every row of the wavefront, from cur0 and cur1, and the scores of the next tile.  An
    // instruction that needs the result of the one before it waits twice as long as any other: four scores at a time go
    // through difference, product and exponential, and a slot later into the sums.
    auto pass1_tile = [&](int T, const agq_v16i &cur0, const agq_v16i &cur1, agq_v16i &nxt0, agq_v16i &nxt1) {
        const uint8_t *const ahead = kt + ((T + 1) & (kRing - 1)) * kKTile;
        copy_k();
#pragma unroll
        for (int s = 0; s < DT; ++s) read_k(s, ahead, 0);
        int mx[4] = {run_m + kBias, cur0[0], cur1[0], cur0[1]};
#pragma unroll
        for (int r = 0; r < 16; ++r) mx[r & 3] = max(mx[r & 3], max(cur0[r], cur1[r]));
        const int nm = max(max(mx[0], mx[1]), max(mx[2], mx[3])) - kBias;
        // kappa s - kappa M with one rounding, that of kappa M, or kappa (s - M) (WIDE)
        const float ref = WIDE ? AGQ_MAGIC + (float)nm : AGQ_MAGIC, nmf = WIDE ? 0.f : -kappa * (float)nm;
        const float keep = __builtin_amdgcn_exp2f(kappa * (float)(run_m - nm));
        float add0 = 0.f, add1 = 0.f;
        constexpr int R = 16 / DT;                               // scores of a slot: R / 2 of either sub-tile
        float e[R];
        auto slot = [&](auto k_tag) {
            constexpr int k = decltype(k_tag)::value, s = k % DT;
            if constexpr (k < 2 * DT) {
                mfma_s(s, k < DT ? nxt0 : nxt1);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (k < DT) read_k(s, ahead, 1);
                float x[R];
#pragma unroll
                for (int r = 0; r < R; ++r) x[r] = __int_as_float(r & 1 ? cur1[k * (R / 2) + r / 2] : cur0[k * (R / 2) + r / 2]) - ref;
                __builtin_amdgcn_sched_barrier(0);
                if (k > 0) {
#pragma unroll
                    for (int r = 0; r < R; ++r) (r & 1 ? add1 : add0) += e[r];
                }
#pragma unroll
                for (int r = 0; r < R; ++r) x[r] = scaled(x[r], nmf);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int r = 0; r < R; ++r) e[r] = __builtin_amdgcn_exp2f(x[r]);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        slot(Int<0>{}); slot(Int<1>{}); slot(Int<2>{}); slot(Int<3>{}); slot(Int<4>{}); slot(Int<5>{}); slot(Int<6>{}); slot(Int<7>{});
#pragma unroll
        for (int r = 0; r < R; ++r) (r & 1 ? add1 : add0) += e[r];
        run_s = run_s * keep + (add0 + add1);
        run_m = nm;
        meet<kKC>();                                             // the tile after the next one has landed
    };
    int T = 0;
    for (; T + 2 <= n_main; T += 2) {
        pass1_tile(T, acc0, acc1, acc2, acc3);
        pass1_tile(T + 1, acc2, acc3, acc0, acc1);
    }
    auto last_tile = [&](int T, const agq_v16i &cur0, const agq_v16i &cur1) {
        const int sub = 2 * T;
        if (sub + 1 < last_sub) {
            tile_stats(cur0, cur1);
        } else {
            if (sub <= last_sub) stats(cur0, sub, sub == last_sub);
            if (sub + 1 <= last_sub) stats(cur1, sub + 1, true);
        }
    };
    if (a.causal) {                                              // the two tiles at the diagonal
        copy_k();
        tile_scores(kt + ((T + 1) & (kRing - 1)) * kKTile, acc2, acc3);
        last_tile(T, acc0, acc1);
        meet<kKC>();
        copy_k();
        last_tile(T + 1, acc2, acc3);
        meet<kKC>();
    }
    // the two lanes of a query (k-groups 0 and 1) join their halves; every row has its own key, so M is a real score
    const int om = __shfl_xor(run_m, 32);
    const float os = __shfl_xor(run_s, 32);
    const int M = max(run_m, om);
    // (a half with nothing counted has sum 0, whatever its factor)
    const float tot = run_s * __builtin_amdgcn_exp2f(kappa * (float)(run_m - M)) +
                      os * __builtin_amdgcn_exp2f(kappa * (float)(om - M));
    // -log2 p = t = kappa (M - s) + log2(tot).  The weight 2^(qmax - c) has the fp16 exponent field
    // 15 + qmax - c = round(15 + qmax - t) clamped to [15, 15 + qmax]: one fused multiply-add gives 15 + qmax - t, and
    // a conversion to a byte rounds it (to even: a tie has measure zero and lies inside the evaluation error anyway) and cuts
    // it off at 0; the lower bound of 15 follows on the weights' patterns, two at a time.  (A dead key's byte may exceed
    // 15 + qmax; what it shifts into the next byte stays among dead keys, whose weights and codes are masked.)
    const float c1 = (float)(15 + a.qmax) - __builtin_amdgcn_logf(tot);                       // v_log_f32: base 2
    const float c2 = WIDE ? c1 : c1 - kappa * (float)M;
    const float zero = WIDE ? AGQ_MAGIC + (float)M : AGQ_MAGIC;
    auto score_of = [&](int bits) { return __int_as_float(bits) - zero; };                    // WIDE: its difference to M

    // ---- pass 2: codes, weights, product with V
    agq_v16f acc_o[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc_o[n][r] = 0.f;
    uint32_t v_rd[4];                                            // operand reads: chunk 4 sub + 2 u + g of row c
#pragma unroll
    for (int i = 0; i < 4; ++i) v_rd[i] = (uint32_t)(c * 128 + (((2 * i + g) ^ ((c >> 1) & 7)) << 4));
    agq_v8h vf[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) vf[n] = agq_v8h{};
    uint32_t f0 = 0, f1 = 0;                                     // exponents of a half sub-tile's eight weights, a byte each
    agq_u4 w;

    {
        const uint8_t *const first = kt + (nt & (kRing - 1)) * kKTile;
#pragma unroll
        for (int s = 0; s < DT; ++s) read_k(s, first, 0);
        read_v(0);
#pragma unroll
        for (int s = 0; s < DT; ++s) mfma_s(s, acc0);
#pragma unroll
        for (int s = 0; s < DT; ++s) read_k(s, first, 1);
        store_v(0, Int<0>{});
        store_v(0, Int<1>{});
        if constexpr (NB == 4) {
            store_v(0, Int<2>{});
            store_v(0, Int<3>{});
        }
    }
    // importance on the quantized map: the weight of the first key (always live)
    if (a.score && g == 0)
        atomicAdd(&a.score[row], 1 << (max(__builtin_amdgcn_cvt_pk_u8_f32(fmaf(kappa, score_of(acc0[0]), c2), 0, 0), 15u) - 15u));
    meet<63>();                                                  // V tile 0 is in LDS

    // the weights of half sub-tile `hs` (keys 16 hs ..) from their exponents
    auto exponents = [&] {                                       // upper bytes of the fp16 patterns
        f0 <<= 2;
        f1 <<= 2;
    };
    auto weights = [&](int hs, auto masked_tag) {
        constexpr bool MASKED = decltype(masked_tag)::value;
        auto two = [](uint32_t f, uint32_t sel) {                // two bytes as upper bytes of two patterns, not below 2^0
            typedef unsigned short us2 __attribute__((ext_vector_type(2)));
            return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(us2, __builtin_amdgcn_perm(f, f, sel)), us2{0x3C00, 0x3C00}));
        };
        w[0] = two(f0, 0x010C000Cu);
        w[1] = two(f0, 0x030C020Cu);
        w[2] = two(f1, 0x010C000Cu);
        w[3] = two(f1, 0x030C020Cu);
        if (MASKED) {
            const int left = row - (16 * hs + 4 * g);            // key i of a lane's four is live if i <= left
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int key = 8 * (i >> 1) + 2 * (i & 1);
                w[i] &= (key <= left ? 0xFFFFu : 0u) | (key + 1 <= left ? 0xFFFF0000u : 0u);
            }
        }
    };
    auto codes = [&](int hs, uint32_t f, int q, auto masked_tag) {   // keys 16 hs + 8 q + 4 g .. + 3
        const int key = 16 * hs + 8 * q + 4 * g;
        uint32_t cw = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            cw |= ((decltype(masked_tag)::value && key + r > row) ? (uint32_t)a.qmax : 15u + (uint32_t)a.qmax - max((f >> (8 * r)) & 255u, 15u)) << (4 * r);
        *reinterpret_cast<uint16_t *>(a.codes + ((int64_t)h * S + row) * (S >> 1) + (key >> 1)) = (uint16_t)cw;
    };
    // Half a sub-tile (16 keys: registers 8 u .. 8 u + 7 of the scores): the exponents of its weights, the product of the half
    // before it with V, and half of the scores of the next sub-tile, dealt out one MFMA at a time.  The eight scores go
    // through conversion, product and rounding in pairs, a slot for each, so that no instruction needs the result of
    // one right before it.  `other` is run in the slots.
    auto half = [&](const agq_v16i &cur, agq_v16i &nxt, int sub, auto u_tag, const uint8_t *vtile, const uint8_t *ahead, auto masked_tag, auto other) {
        constexpr int u = decltype(u_tag)::value;
        const int vi = 2 * (sub & 1) + u, hs = 2 * sub + u;
        // of a sub-tile with dead keys no other follows, so the half before this one has some only if it is the same sub-tile's
        const std::integral_constant<bool, decltype(masked_tag)::value && u == 1> before_tag{};
        float x[8];
        uint32_t n0 = 0, n1 = 0;
        auto cvt = [&](auto i_tag) {                             // pair i: registers i and i + 4
            constexpr int i = decltype(i_tag)::value;
            x[i] = score_of(cur[8 * u + i]);
            x[i + 4] = score_of(cur[8 * u + i + 4]);
        };
        auto mul = [&](auto i_tag) {
            constexpr int i = decltype(i_tag)::value;
            x[i] = fmaf(kappa, x[i], c2);
            x[i + 4] = fmaf(kappa, x[i + 4], c2);
        };
        auto rnd = [&](auto i_tag) {
            constexpr int i = decltype(i_tag)::value;
            n0 = __builtin_amdgcn_cvt_pk_u8_f32(x[i], i, n0);
            n1 = __builtin_amdgcn_cvt_pk_u8_f32(x[i + 4], i, n1);
        };
        auto pv = [&](auto n_tag) {
            constexpr int n = decltype(n_tag)::value;
            acc_o[n] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(agq_v8h, w), vf[n], acc_o[n], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            vf[n] = *reinterpret_cast<const agq_v8h *>(vtile + v_rd[vi] + n * (32 * 128));
        };
        auto qk = [&](auto s_tag) {
            constexpr int s = decltype(s_tag)::value;
            mfma_s(s, nxt);
            __builtin_amdgcn_sched_barrier(0);
            read_k(s, ahead, sub & 1);
        };
        auto end_slot = [&](auto k_tag) {
            other(k_tag);
            __builtin_amdgcn_sched_barrier(0);
        };
        constexpr Int<0> i0; constexpr Int<1> i1; constexpr Int<2> i2; constexpr Int<3> i3; constexpr Int<4> i4; constexpr Int<5> i5;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (NB == 4) {
            qk(Int<2 * u>{});
            exponents(); cvt(i0); weights(hs - 1, before_tag);
            end_slot(i0);
            pv(i0);
            cvt(i1); mul(i0);
            end_slot(i1);
            pv(i1);
            cvt(i2); mul(i1); rnd(i0);
            end_slot(i2);
            qk(Int<2 * u + 1>{});
            cvt(i3); mul(i2); rnd(i1);
            end_slot(i3);
            pv(i2);
            mul(i3); rnd(i2);
            end_slot(i4);
            pv(i3);
            rnd(i3);
            end_slot(i5);
        } else {
            qk(Int<u>{});
            exponents(); cvt(i0); cvt(i1); weights(hs - 1, before_tag);
            end_slot(i0);
            pv(i0);
            cvt(i2); cvt(i3); mul(i0); mul(i1); rnd(i0);
            end_slot(i1);
            pv(i1);
            mul(i2); mul(i3); rnd(i1); rnd(i2); rnd(i3);
            end_slot(i2);
        }
        f0 = n0;
        f1 = n1;
        if (CODES) {
            codes(hs, f0, 0, masked_tag);
            codes(hs, f1, 1, masked_tag);
        }
    };
    auto pass2_tile = [&](int t, auto masked_tag) {
        constexpr bool MASKED = decltype(masked_tag)::value;
        const uint8_t *const vtile = vt + (t & 1) * kVTile;
        const uint8_t *const ahead = kt + ((nt + t + 1) & (kRing - 1)) * kKTile;
        auto none = [](auto) {};
        auto stage = [&](auto part_tag) {                        // the V tile t + 1, a part of its rows
            constexpr int part = decltype(part_tag)::value;
            if constexpr (NB == 4) store_v(t + 1, part_tag);
            else if constexpr ((part & 1) == 0) store_v(t + 1, Int<part / 2>{});
        };
        constexpr int kAt = NB == 4 ? 4 : 2;                     // slot that does it
#define AGQ_STAGE(P)                                                     \
    [&](auto k) {                                                        \
        if constexpr (decltype(k)::value == kAt) stage(Int<P>{});        \
        if constexpr (decltype(k)::value == 1 && P == 1) copy_v();  \
        if constexpr (decltype(k)::value == 1 && P == 2) copy_k(); \
    }
        if (!MASKED || t + 1 < nt) read_v(t + 1);
        if constexpr (!MASKED) {
            half(acc0, acc1, 2 * t, Int<0>{}, vtile, ahead, masked_tag, AGQ_STAGE(0));
            half(acc0, acc1, 2 * t, Int<1>{}, vtile, ahead, masked_tag, AGQ_STAGE(1));
            half(acc1, acc0, 2 * t + 1, Int<0>{}, vtile, ahead, masked_tag, AGQ_STAGE(2));
            half(acc1, acc0, 2 * t + 1, Int<1>{}, vtile, ahead, masked_tag, AGQ_STAGE(3));
        } else {
            if (t + 1 < nt) {
                stage(Int<0>{});
                stage(Int<1>{});
                stage(Int<2>{});
                stage(Int<3>{});
            }
            if (2 * t <= last_sub) {
                half(acc0, acc1, 2 * t, Int<0>{}, vtile, ahead, masked_tag, none);
                half(acc0, acc1, 2 * t, Int<1>{}, vtile, ahead, masked_tag, none);
            }
            if (2 * t + 1 <= last_sub) {
                half(acc1, acc0, 2 * t + 1, Int<0>{}, vtile, ahead, masked_tag, none);
                half(acc1, acc0, 2 * t + 1, Int<1>{}, vtile, ahead, masked_tag, none);
            }
        }
#undef AGQ_STAGE
        if constexpr (!MASKED) meet<kKC>();                      // V tile t + 2 and K tile nt + t + 2 have landed
        else if (t + 1 < nt) meet<63>();                         // the last V tile is in LDS; no more are copied (nor waited for: 7.22 -> 6.85)
    };
    int t = 0;
    for (; t < n_main; ++t) pass2_tile(t, std::false_type{});
    for (; t < nt; ++t) pass2_tile(t, std::true_type{});
    exponents();
    if (a.causal) weights(2 * last_sub + 1, std::true_type{});
    else weights(0, std::false_type{});
#pragma unroll
    for (int n = 0; n < NB; ++n) acc_o[n] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(agq_v8h, w), vf[n], acc_o[n], 0, 0, 0);

    __builtin_amdgcn_s_waitcnt(0x70);                            // the last copies into LDS have landed before it is given back

    // code map right of the last sub-tile this wavefront multiplied: all qmax
    if (CODES && a.causal) {
        const uint32_t fill = 0x11111111u * (uint32_t)a.qmax;
        uint8_t *dst = a.codes + ((int64_t)h * S + row) * (S >> 1);
        for (int k = (last_sub + 1) * 32 + g * 8; k < S; k += 16) *reinterpret_cast<uint32_t *>(dst + (k >> 1)) = fill;
    }

    // accumulator register 4 q + r holds query row 8 q + 4 g + r of the wavefront,
    // channel NB c + n in block n: NB consecutive channels per lane and row
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int orow = r0 + 8 * q + 4 * g + r;
            uint32_t hv[NB / 2];
#pragma unroll
            for (int n = 0; n < NB; n += 2)
                hv[n / 2] = __half_as_ushort(__float2half_rn(acc_o[n][4 * q + r] * a.out_scale)) |
                            (uint32_t)__half_as_ushort(__float2half_rn(acc_o[n + 1][4 * q + r] * a.out_scale)) << 16;
            uint32_t *const dst = reinterpret_cast<uint32_t *>(a.o + (int64_t)orow * ((int64_t)H * D) + (int64_t)h * D + NB * c);
            if constexpr (NB == 4) *reinterpret_cast<uint2 *>(dst) = make_uint2(hv[0], hv[1]);
            else *dst = hv[0];
            if constexpr (TILES) {
                uint32_t code[NB];
#pragma unroll
                for (int n = 0; n < NB; ++n)
                    code[n] = agq_quant1(__half2float(__ushort_as_half((unsigned short)(hv[n / 2] >> (16 * (n & 1))))), a.quant);
                const int ch = h * D + NB * c;
                char *const at = a.tiles + agq_code_offset(orow, ch >> 3, H * D >> 7) + (ch & 7);
                if constexpr (NB == 4) *reinterpret_cast<uint32_t *>(at) = agq_pack4(code[0], code[1], code[2], code[3]);
                else *reinterpret_cast<uint16_t *>(at) = (uint16_t)((code[0] & 255u) | (code[1] << 8));
            }
        }
}

}  // namespace

int agq_launch_qk_log2_attn(const int8_t *q, const int8_t *k, const int8_t *v, int64_t H, int64_t S, int64_t D, int causal,
                            int qmax, int e_q, int e_k, int e_v, void *o, void *codes, int32_t *score, const AgqCodes &o_codes, void *stream) {
    QkArgs a;
    a.q = q;
    a.k = k;
    a.v = v;
    a.o = (__half *)o;
    a.codes = (uint8_t *)codes;
    a.score = score;
    a.H = (int)H;
    a.S = (int)S;
    a.causal = causal;
    a.qmax = qmax;
    a.kappa = (float)(ldexp(1.0, e_q + e_k) * 1.4426950408889634 / sqrt((double)D));
    a.out_scale = ldexpf(1.0f, e_v - qmax + 9);
    a.tiles = (char *)o_codes.tiles;
    a.quant = o_codes.tiles ? agq_make_quant_signed(o_codes.bits, o_codes.e, 0) : AgqQuant{};
    static int ncu_of[64] = {0};
    int device = 0;
    if (hipGetDevice(&device) != hipSuccess) return (int)hipGetLastError();
    int ncu = (device >= 0 && device < 64) ? ncu_of[device] : 0;
    if (ncu == 0) {
        if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || ncu < 1) ncu = 256;
        if (device >= 0 && device < 64) ncu_of[device] = ncu;
    }
    a.ncu = ncu;
    hipStream_t st = (hipStream_t)stream;
    const unsigned grid = (unsigned)((S / kQRows) * H);
    auto launch = [&](auto kernel) { kernel<<<grid, 256, 0, st>>>(a); };
    auto pick = [&](auto dt_tag, auto wide_tag) {
        constexpr int DT = decltype(dt_tag)::value;
        constexpr bool WIDE = decltype(wide_tag)::value;
        if (codes) launch(qk_log2_attn_kernel<DT, true, false, WIDE>);
        else if (a.tiles) launch(qk_log2_attn_kernel<DT, false, true, WIDE>);
        else launch(qk_log2_attn_kernel<DT, false, false, WIDE>);
    };
    if (D == 128) a.kappa > 1.0f ? pick(Int<4>{}, std::true_type{}) : pick(Int<4>{}, std::false_type{});
    else a.kappa > 1.0f ? pick(Int<2>{}, std::true_type{}) : pick(Int<2>{}, std::false_type{});
    return (int)hipGetLastError();
}
