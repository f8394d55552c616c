// Log2-quantized softmax probabilities times the int8 value matrix, the
// start-token importance score, and token pruning.
//
// Eq.3 (Section 4.1) on a probability p = 2^E (1 + f) needs no logarithm:
// round(-log2 p) = -E when 1 + f < sqrt(2) and -E - 1 otherwise, and
// -log2 p is never half-way between integers for a rational p.  On fp16 bit
// patterns h (normal numbers) this is 15 - ((h + 599) >> 10): 1 + 425/1024 is
// the first mantissa above sqrt(2), and adding 1024 - 425 carries into the
// exponent field exactly from there on.  Subnormals (h < 1024, value h * 2^-24)
// round to 14 from h = 725 on, else to 15 or more.
//
// The product uses the fp16 MFMA with fp32 accumulation on the integers
// 2^(qmax - c) and v: every term and every partial sum is an integer below
// 2^24 for softmax rows, so the result is exact in any order.
#include "agq_device.h"
#include "agq_internal.h"

AgqQuant agq_make_quant_signed(int bits, int e, int zp);   // agq_quant.hip

#include <type_traits>

typedef _Float16 agq_v8h __attribute__((ext_vector_type(8)));
typedef _Float16 agq_v2h __attribute__((ext_vector_type(2)));
typedef unsigned short agq_v2us __attribute__((ext_vector_type(2)));
typedef float agq_v16f __attribute__((ext_vector_type(16)));
typedef uint32_t agq_u4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int kQRows = 128;     // query rows per workgroup (32 per wavefront)
constexpr int kKeys = 64;       // keys per tile: four MFMA steps of 16
constexpr int kVRow = 144;      // bytes per channel row of the V tile in LDS: 64 keys in fp16 + 16 of padding
constexpr int kMaxD = 256;

struct AttnArgs {
    const uint16_t *p;   // fp16 bits [H,S,S]
    const int8_t *v;     // [H,S,D]
    __half *o;           // [S, H*D]
    uint8_t *codes;      // [H,S,S/2] or null
    int32_t *score;      // [S] or null
    int H, S, D;
    int causal, qmax;
    float out_scale;     // 2^(e_v - qmax)
    int ncu;             // compute units of the device (ordering of the causal row blocks)
};

// Two probabilities (packed fp16) -> two weights 2^(qmax - c) as packed fp16 bit
// patterns.  Scaling by 2^10 first makes every non-zero input a normal number, so
// one formula covers subnormals: with e = (bits(1024 p) + 599) >> 10 the code is
// c = min(25 - e, qmax) and the weight's exponent field 15 + max(e - (25 - qmax), 0).
// kmin = (25 - qmax) << 10 and kadd = (qmax - 10) << 10, both replicated per half
// (kadd in wrap-around arithmetic: no half ever borrows from the other).
__device__ __forceinline__ uint32_t log2_weight2(uint32_t p2, uint32_t kmin, uint32_t kadd) {
    const agq_v2h x = __builtin_bit_cast(agq_v2h, p2) * agq_v2h{(_Float16)1024.0f, (_Float16)1024.0f};
    uint32_t u = (__builtin_bit_cast(uint32_t, x) + 0x02570257u) & 0xFC00FC00u;
    agq_v2us e = __builtin_bit_cast(agq_v2us, u);
    e = __builtin_elementwise_min(__builtin_elementwise_max(e, __builtin_bit_cast(agq_v2us, kmin)),
                                  agq_v2us{25u << 10, 25u << 10});
    return __builtin_bit_cast(uint32_t, e) + kadd;
}

// Byte offset of the 16-byte piece (eight keys in fp16) `chunk` of row `slot`
// inside the LDS tile; rows are padded to 144 bytes so that sixteen lanes
// reading the same chunk of consecutive rows hit sixteen different bank groups.
__device__ __forceinline__ int vt_offset(int slot, int chunk) { return slot * kVRow + (chunk << 4); }

// One workgroup = 128 query rows of one head; wavefront w owns rows 32 w .. 32 w + 31
// as the A operand of the 32x32x16 fp16 MFMA (lane: row l & 31, eight keys of
// k-group l >> 5).  Inside a 64-key tile the keys are dealt to the MFMA steps so
// that a lane's four steps cover 32 consecutive keys (64 contiguous bytes of its
// row): step t of k-group g uses keys 32 g + 8 t .. + 7, for both operands.
// V tile: int8 [key][d] -> fp16 [d][key] in LDS, once per workgroup and tile.  A
// thread unit is (eight keys, four channels): eight dword loads, a byte
// transpose by v_perm that puts each byte u = v + 128 under 0x64 (the fp16
// pattern of 1024 + u), minus 1152, four 16-byte LDS writes.  Channel d sits in
// row (d & 3) * D/4 + (d >> 2), so the conversion writes and the MFMA reads both
// walk consecutive rows, and a lane ends up with four consecutive channels of
// its query rows.
// P runs two tiles ahead in registers, V one tile ahead; V loads are issued
// before the P loads so that waiting for V leaves the P loads in flight.
template <int CB, bool CODES>
__global__ __launch_bounds__(256, CB == 1 ? 3 : 1) void log2_attn_kernel(const AttnArgs a) {
    constexpr int NBUF = CB == 1 ? 2 : 1;
    __shared__ __align__(16) uint8_t vt[NBUF][CB * 128 * kVRow];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int S = a.S, D = a.D, H = a.H, DQ = D >> 2;
    const int nb = (S + kQRows - 1) / kQRows;

    // workgroup -> (head, row block).  Causal: blocks ranked by length, longest first.
    // All workgroups of a launch are resident at once when there are at most three
    // per CU, and the dispatcher hands workgroup i and workgroup i + (number of CUs)
    // to the same CU; every second run of that many workgroups therefore takes its
    // blocks in ascending order, so that a CU's long first block is paired with a
    // short second one and the CUs finish together (loads of 19-24 instead of 14-30
    // units at H = 40, S = 2048).
    int rank = (int)blockIdx.x;
    if (a.causal) {
        const int run = rank / a.ncu, base = run * a.ncu;
        if (run & 1) rank = base + min(a.ncu, (int)gridDim.x - base) - 1 - (rank - base);
    }
    const int h = rank % H;
    const int b = a.causal ? nb - 1 - rank / H : rank / H;
    const int q0 = b * kQRows;
    const int r0 = q0 + wave * 32;                        // first row of this wavefront
    const int row = r0 + (lane & 31);
    const int g = lane >> 5;
    const int last_key = a.causal ? min(q0 + kQRows, S) : S;
    const int nt = (last_key + kKeys - 1) / kKeys;
    // Step t of this workgroup handles tile (t + rot) mod nt.  Workgroups that run
    // side by side would otherwise all read the same column window of their rows
    // at the same time; with a row pitch that is a power of two those addresses
    // fall on few memory channels.
    const int rot = (int)((blockIdx.x * 11u) % (unsigned)nt);
    auto tile_of = [&](int t) {
        int kt = min(t, nt - 1) + rot;
        return kt >= nt ? kt - nt : kt;
    };
    const int lim = a.causal ? row : S - 1;               // last key this row uses
    const int wave_lim = a.causal ? r0 : S - 1;           // a tile reaching past this needs the mask
    const int wave_last = a.causal ? r0 + 31 : S - 1;     // tiles starting past this are dead for the wavefront

    const uint32_t kmin = ((uint32_t)(25 - a.qmax) << 10) * 0x00010001u;
    const uint32_t kadd = (uint32_t)((a.qmax - 10) * 1024) * 0x00010001u;
    const uint32_t ctop = ((uint32_t)(15 + a.qmax) << 10) * 0x00010001u;
    const uint32_t cdead = ((uint32_t)a.qmax << 10) * 0x00010001u;

    // Addresses are a uniform base plus a 32-bit per-lane byte offset (one head of
    // P is below 4 GiB: S <= 32768).
    const uint8_t *phead = reinterpret_cast<const uint8_t *>(a.p + (int64_t)h * S * S);
    const uint32_t prow_off = (uint32_t)min(row, S - 1) * (uint32_t)S * 2u;
    // V conversion units of this thread: (eight keys kg, four channels 4 c .. 4 c + 3)
    uint32_t vraw[CB][8];
    int vu_c[CB], vu_kg[CB];
    bool vu_ok[CB];
#pragma unroll
    for (int u = 0; u < CB; ++u) {
        const int unit = threadIdx.x + 256 * u;
        vu_ok[u] = unit < 8 * DQ;
        vu_c[u] = unit % DQ;
        vu_kg[u] = vu_ok[u] ? unit / DQ : 0;
    }
    const int8_t *vh = a.v + (int64_t)h * S * D;
    auto load_v = [&](int t) {
        const int k0 = tile_of(t) * kKeys;
#pragma unroll
        for (int u = 0; u < CB; ++u)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int key = min(k0 + 8 * vu_kg[u] + i, S - 1);   // keys past S get weight 0
                vraw[u][i] = *reinterpret_cast<const uint32_t *>(vh + (uint32_t)(key * D + 4 * vu_c[u]));
            }
    };
    auto store_v = [&](uint8_t *buf) {
        const agq_v2h bias = {(_Float16)1152.0f, (_Float16)1152.0f};
#pragma unroll
        for (int u = 0; u < CB; ++u) {
            uint32_t x[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = vraw[u][i] ^ 0x80808080u;     // bytes v + 128
#pragma unroll
            for (int bb = 0; bb < 4; ++bb) {
                // halves 0x64uu = 1024 + (v + 128) of keys 2 i and 2 i + 1 of channel 4 c + bb
                const uint32_t sel = 0x0C000C00u | (uint32_t)bb | ((uint32_t)(4 + bb) << 16);
                agq_u4 out;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t w = __builtin_amdgcn_perm(x[2 * i + 1], x[2 * i], sel) | 0x64006400u;
                    out[i] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(agq_v2h, w) - bias);
                }
                if (vu_ok[u]) *reinterpret_cast<agq_u4 *>(buf + vt_offset(bb * DQ + vu_c[u], vu_kg[u])) = out;
            }
        }
    };
    // four 16-byte pieces of this lane's row: keys k0 + 32 g + 8 t .. + 7
    auto load_p = [&](agq_u4 (&dst)[4], int t) {
        int tt = tile_of(t);
        if (tt * kKeys > wave_last) tt = 0;               // dead tile: re-read a line that is already cached
#pragma unroll
        for (int st = 0; st < 4; ++st) {
            const uint32_t kc = (uint32_t)min(tt * kKeys + 32 * g + 8 * st, S - 8);
            dst[st] = *reinterpret_cast<const agq_u4 *>(phead + (prow_off + kc * 2u));
        }
    };

    agq_v16f acc[4][CB];
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[n][cb][r] = 0.f;

    __shared__ int ssum[kQRows];
    if (a.score && threadIdx.x < kQRows) ssum[threadIdx.x] = 0;   // made visible by the main loop's barriers

    int bslot[CB];                                          // LDS row of this lane's B operand, n = 0
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) bslot[cb] = min(cb * 32 + (lane & 31), DQ - 1);

    // MASKED: the tile reaches past the last key of some row (diagonal tiles of the
    // causal case, the ragged last tile); dead keys get weight 0 and code qmax.
    auto multiply = [&](const agq_u4 (&pc)[4], int k0, const uint8_t *buf, auto masked_tag) {
        constexpr bool MASKED = decltype(masked_tag)::value;
#pragma unroll
        for (int st = 0; st < 4; ++st) {
            const int kc = k0 + 32 * g + 8 * st;
            const int nl = lim - kc + 1;                   // live keys of this piece (may be <= 0 or >= 8)
            uint32_t wv[4];
            uint32_t cw = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                uint32_t u = log2_weight2(pc[st][j], kmin, kadd);
                uint32_t m = 0xFFFFFFFFu;
                if (MASKED) {
                    const int lv = nl - 2 * j;
                    m = lv >= 2 ? 0xFFFFFFFFu : (lv == 1 ? 0x0000FFFFu : 0u);
                    u &= m;
                }
                if (CODES) {
                    uint32_t c10 = ctop - u;               // code << 10 per half (dead: above qmax, fixed below)
                    if (MASKED) c10 = (c10 & m) | (cdead & ~m);
                    cw |= (((c10 >> 10) | (c10 >> 22)) & 0xFFu) << (8 * j);
                }
                wv[j] = u;
            }
            if (CODES) {
                if (row < S && kc < S)
                    *reinterpret_cast<uint32_t *>(a.codes + ((int64_t)h * S + row) * (S >> 1) + (kc >> 1)) = cw;
            }
            const agq_u4 wq = {wv[0], wv[1], wv[2], wv[3]};
            const agq_v8h af = __builtin_bit_cast(agq_v8h, wq);
#pragma unroll
            for (int n = 0; n < 4; ++n)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) {
                    const int slot = n * DQ + bslot[cb];
                    const agq_v8h bf = *reinterpret_cast<const agq_v8h *>(buf + vt_offset(slot, 4 * g + st));
                    acc[n][cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(af, bf, acc[n][cb], 0, 0, 0);
                }
        }
    };
    auto compute = [&](const agq_u4 (&pc)[4], int t, const uint8_t *buf) {
        const int k0 = tile_of(t) * kKeys;
        if (k0 > wave_last) return;
        if (k0 + kKeys - 1 > wave_lim) multiply(pc, k0, buf, std::true_type{});
        else multiply(pc, k0, buf, std::false_type{});
    };

    // tile t: V(t) registers -> LDS, issue V(t+1) then P(t+2), barrier, multiply
    auto tile = [&](const agq_u4 (&pc)[4], agq_u4 (&pfar)[4], int t, bool more_v, bool more_p) {
        uint8_t *buf = vt[NBUF == 2 ? (t & 1) : 0];
        if (NBUF == 1) __syncthreads();                     // everyone is done reading the only buffer
        store_v(buf);
        if (more_v) load_v(t + 1);
        if (more_p) load_p(pfar, t + 2);
        __syncthreads();
        compute(pc, t, buf);
    };

    // The steady-state loop always runs three whole tiles, so every path around
    // its back edge has consumed the same register sets; the last one or two
    // tiles follow outside it.
    agq_u4 p0[4], p1[4], p2[4];
    load_v(0);
    load_p(p0, 0);
    load_p(p1, 1);
    int t = 0;
    for (; t + 3 <= nt; t += 3) {
        tile(p0, p2, t, true, true);
        tile(p1, p0, t + 1, true, true);
        tile(p2, p1, t + 2, true, true);
    }
    if (t < nt) {
        const bool two = t + 2 == nt;                       // uniform over the workgroup
        tile(p0, p2, t, true, false);
        if (two) tile(p1, p0, t + 1, false, false);
    }

    // code map right of the last tile this wavefront multiplied: all qmax
    if (CODES && a.causal && row < S) {
        const uint32_t fill = 0x11111111u * (uint32_t)a.qmax;
        uint8_t *dst = a.codes + ((int64_t)h * S + row) * (S >> 1);
        const int done = min(nt, wave_last / kKeys + 1);
        for (int k = done * kKeys + g * 8; k < S; k += 16) *reinterpret_cast<uint32_t *>(dst + (k >> 1)) = fill;
    }

    // accumulator register 4 q + r holds query row 8 q + 4 g + r of the wavefront,
    // channel 4 c + n in tile n: four consecutive channels per lane and row
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
        const int c = cb * 32 + (lane & 31);
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int orow = r0 + 8 * q + 4 * g + r;
                __half hv[4];
#pragma unroll
                for (int n = 0; n < 4; ++n) hv[n] = __float2half_rn(acc[n][cb][4 * q + r] * a.out_scale);
                if (orow < S && c < DQ)
                    *reinterpret_cast<uint2 *>(a.o + (int64_t)orow * ((int64_t)H * D) + (int64_t)h * D + 4 * c) =
                        *reinterpret_cast<const uint2 *>(hv);
            }
    }

    // Importance of a token = attention it pays to the first token, summed over
    // heads as exact integers p * 2^24 (Section 4.3).  The 128 rows of a row block
    // are dealt to the H workgroups that share it; each loads its rows' first
    // column from every head (one value per thread) and sums them in LDS.
    if (a.score) {
        const int rows_per = (kQRows + H - 1) / H;
        const int j = threadIdx.x / H, hh = threadIdx.x - j * H;
        const int i = q0 + h * rows_per + j;
        if (j < rows_per && h * rows_per + j < kQRows && i < S)
            atomicAdd(&ssum[j], (int)(__half2float(__ushort_as_half(a.p[((int64_t)hh * S + i) * S])) * 16777216.0f));
        __syncthreads();
        const int io = q0 + h * rows_per + (int)threadIdx.x;
        if ((int)threadIdx.x < rows_per && h * rows_per + (int)threadIdx.x < kQRows && io < S)
            a.score[io] = ssum[threadIdx.x];
    }
}

// ------------------------------------------------------------------ pruning

constexpr int kSelMaxS = 8192;
constexpr int kSelChunks = kSelMaxS / 64;

// One cross-lane step in the data path of the vector ALU; lanes without a source contribute 0.
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ uint32_t dpp0(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ uint32_t wave_or(uint32_t v) {          // uniform
    v |= dpp0<0xB1>(v);                                            // quads, halves of eight, of sixteen
    v |= dpp0<0x4E>(v);
    v |= dpp0<0x141>(v);
    v |= dpp0<0x140>(v);
    return __builtin_amdgcn_readlane(v, 0) | __builtin_amdgcn_readlane(v, 16) | __builtin_amdgcn_readlane(v, 32) | __builtin_amdgcn_readlane(v, 48);
}
__device__ __forceinline__ int wave_scan(int x) {                  // inclusive sum over lanes
    uint32_t v = (uint32_t)x;
    v += dpp0<0x111>(v);                                           // shifted right by 1, 2, 4, 8 within sixteen lanes
    v += dpp0<0x112>(v);
    v += dpp0<0x114>(v);
    v += dpp0<0x118>(v);
    v += dpp0<0x142, 0xA>(v);                                      // lane 15 to the second and fourth sixteen
    v += dpp0<0x143, 0xC>(v);                                      // lane 31 to the upper half
    return (int)v;
}

// Output row p from src, the chunks c, c + stride, ...; with CODES the row's Eq.2 codes as well.
template <bool CODES>
__device__ __forceinline__ void copy_row(const uint4 *__restrict__ src, uint4 *__restrict__ dst, int p, int d8, int c, int stride,
                                         const AgqQuant &q, char *__restrict__ tiles) {
    const int last = d8 - 1;
    for (; c < d8; c += 4 * stride) {                              // four loads under way at a time
        const uint4 v0 = src[c], v1 = src[min(c + stride, last)], v2 = src[min(c + 2 * stride, last)], v3 = src[min(c + 3 * stride, last)];
        auto put = [&](int at_c, const uint4 &v) {
            if (at_c >= d8) return;
            dst[at_c] = v;
            if (CODES) *reinterpret_cast<uint2 *>(tiles + agq_code_offset(p, at_c, d8 >> 4)) = agq_quant8<true>(v, q);
        };
        put(c, v0);
        put(c + stride, v1);
        put(c + 2 * stride, v2);
        put(c + 3 * stride, v3);
    }
}

// Survivors of Eq.4, the n_keep tokens with the largest score, equal scores to the lower index, in ascending order, and
// their rows: out[p] = x[idx[p]], with CODES also the rows' Eq.2 codes in the operand order of the tiled GEMM.
//
// Every workgroup selects for itself, then copies its few rows: a selection by one workgroup in front of the copies is a
// launch more, and its time is latency whoever does it.  No sort:
//   1. the bits in which scores differ at all, then a radix select of the n_keep-th largest over those (digits of eight
//      bits, histograms in LDS; every wavefront reads the histogram and scans it by itself, with cross-lane
//      operations of the vector ALU, so a digit takes one barrier);
//   2. ballots mark, 64 tokens a word, those above that score and those equal to it, and a second scan over the words
//      gives every word its survivors and their place;
//   3. the token of output row p is then found by a ballot over the words and a search for a set bit.
// Thread t of wavefront w holds the tokens 64 (WAVES e + w) + t.  Against a launch for the selection (one
// workgroup of sixteen wavefronts, four digits always, cross-lane steps through LDS) and one for the rows: 2048 tokens, 1024
// kept, rows of 5120 11.8 -> 8.4 us (14.0 -> 8.8 where scores crowd at one end), 300 tokens, 213 rows of 4096 8.7 -> 4.6,
// 8192 tokens, 4096 rows of 4096 24.0 -> 22.4.  What is left of it: about 2.5 us of latency from the scores to the rows,
// more where a wavefront holds more tokens (code for sixteen tokens a thread alone took 2 us), and the rows.
// WAVES: wavefronts of a workgroup; PER: tokens per thread, in registers.  ROWS: as above; without, one workgroup writes the
// indices alone, which may lie over the scores: every thread holds its own in registers by then.
template <int WAVES, int PER, bool CODES, bool ROWS>
__global__ __launch_bounds__(WAVES * 64) void prune_rows_kernel(const int32_t *score, int S, int n_keep, int rows_per_wg,
                                                                 const uint4 *__restrict__ x, int d8, int32_t *idx_out,
                                                                 uint4 *__restrict__ out, const AgqQuant q, char *__restrict__ tiles) {
    constexpr int kThreads = WAVES * 64;
    __shared__ __align__(16) int hist[4][256];
    __shared__ __align__(16) uint32_t differ[WAVES][2];
    __shared__ __align__(16) uint64_t above_m[kSelChunks], equal_m[kSelChunks];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint32_t key[PER];         // order-preserving unsigned image of the signed score
    uint32_t ones = 0, zeros = 0;
    auto live = [&](int e) { return e * kThreads + tid < S; };
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        key[e] = live(e) ? (uint32_t)score[e * kThreads + tid] ^ 0x80000000u : 0u;
        ones |= key[e];
        zeros |= live(e) ? ~key[e] : 0u;
    }
    for (int i = tid; i < 4 * 256 / 4; i += kThreads) reinterpret_cast<int4 *>(hist)[i] = make_int4(0, 0, 0, 0);
    if (tid < kSelChunks) above_m[tid] = equal_m[tid] = 0;
    ones = wave_or(ones);
    zeros = wave_or(zeros);
    if (lane == 0) {
        differ[wave][0] = ones;
        differ[wave][1] = zeros;
    }
    __syncthreads();
    ones = zeros = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        ones |= differ[w][0];
        zeros |= differ[w][1];
    }
    ones = __builtin_amdgcn_readfirstlane(ones);
    const uint32_t diff = ones & __builtin_amdgcn_readfirstlane(zeros);
    int shift = diff ? 32 - __builtin_clz(diff) : 0;               // bits still to be decided
    uint32_t himask = shift == 32 ? 0u : ~0u << shift, prefix = ones & himask;   // equal in every key
    int k = n_keep;                                                // the k-th largest among the tokens matching `prefix`
    for (int pass = 0; shift > 0; ++pass) {
        shift = max(shift - 8, 0);
        const uint32_t dmask = ~himask >> shift;                   // the digit: eight bits, or what is left
#pragma unroll
        for (int e = 0; e < PER; ++e)
            if (live(e) && (key[e] & himask) == prefix) {
                // the lanes that share the first one's digit add up together: many do where scores crowd at one end
                const uint32_t digit = (key[e] >> shift) & dmask;
                const bool same = digit == __builtin_amdgcn_readfirstlane(digit);
                const uint64_t crowd = __ballot(same);
                if (!same || lane == __builtin_ctzll(crowd)) atomicAdd(&hist[pass][digit], same ? __popcll(crowd) : 1);
            }
        __syncthreads();
        // lane l owns digits 255 - 4 l .. 252 - 4 l: sums over lanes run from the top digit down
        const int4 c = *reinterpret_cast<const int4 *>(&hist[pass][252 - 4 * lane]);
        const int mine = c.x + c.y + c.z + c.w, upto = wave_scan(mine), higher = upto - mine;
        const uint64_t here = __ballot(higher < k && k <= upto);   // one lane: the k-th largest falls into its digits
        const int rem = k - higher, s3 = c.w, s2 = s3 + c.z, s1 = s2 + c.y;
        const int digit = 255 - 4 * lane - (rem > s3) - (rem > s2) - (rem > s1);
        const int left = rem - (rem > s1 ? s1 : rem > s2 ? s2 : rem > s3 ? s3 : 0);
        const int f = __builtin_ctzll(here);
        prefix |= (uint32_t)__builtin_amdgcn_readlane(digit, f) << shift;
        k = __builtin_amdgcn_readlane(left, f);
        himask = shift ? ~0u << shift : ~0u;
    }
    // prefix = image of the n_keep-th largest score; k = number of tokens with exactly that score that survive
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        const uint64_t ab = __ballot(live(e) && key[e] > prefix), eq = __ballot(live(e) && key[e] == prefix);
        if (lane == 0) {
            above_m[e * WAVES + wave] = ab;
            equal_m[e * WAVES + wave] = eq;
        }
    }
    __syncthreads();
    // lane l: words 2 l and 2 l + 1
    const ulonglong2 ab = *reinterpret_cast<const ulonglong2 *>(&above_m[2 * lane]), eq = *reinterpret_cast<const ulonglong2 *>(&equal_m[2 * lane]);
    const int e0 = __popcll(eq.x), e1 = __popcll(eq.y);
    const int ties = wave_scan(e0 + e1) - e0 - e1;                 // equal ones in front of this lane's
    auto lowest = [](uint64_t m, int count, int n) {               // the n lowest of count set bits
        if (n >= count) return m;
        uint64_t rest = m;
        for (; n > 0; --n) rest &= rest - 1;
        return m ^ rest;
    };
    const uint64_t k0 = ab.x | lowest(eq.x, e0, k - ties), k1 = ab.y | lowest(eq.y, e1, k - ties - e0);
    const int n0 = __popcll(k0), n01 = n0 + __popcll(k1), end = wave_scan(n01);

    if constexpr (!ROWS) {
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const int w = e * WAVES + wave, l = w >> 1;            // this wavefront's word lies with lane l
            const uint64_t word = (w & 1) ? k1 : k0;
            const uint64_t kept = ((uint64_t)__builtin_amdgcn_readlane((uint32_t)(word >> 32), l) << 32) | (uint32_t)__builtin_amdgcn_readlane((uint32_t)word, l);
            const int before = __builtin_amdgcn_readlane(end - n01, l) + ((w & 1) ? __builtin_amdgcn_readlane(n0, l) : 0);
            if (kept >> lane & 1) idx_out[before + __popcll(kept & ((1ull << lane) - 1))] = 64 * w + lane;
        }
        return;
    }

    const int per_row = WAVES / rows_per_wg;                   // wavefronts of a row
    for (int p = blockIdx.x * rows_per_wg + wave / per_row; p < n_keep; p += gridDim.x * rows_per_wg) {
        const int f = __builtin_ctzll(__ballot(p < end));              // the first lane whose survivors reach past p
        int r = p - __builtin_amdgcn_readlane(end - n01, f), at = 128 * f;
        const int first = __builtin_amdgcn_readlane(n0, f);
        const bool second = r >= first;
        uint64_t word = second ? k1 : k0;
        uint32_t lo = __builtin_amdgcn_readlane((uint32_t)word, f), hi = __builtin_amdgcn_readlane((uint32_t)(word >> 32), f);
        if (second) {
            r -= first;
            at += 64;
        }
        word = ((uint64_t)hi << 32) | lo;
#pragma unroll
        for (int w = 32; w > 0; w >>= 1) {                             // the r-th set bit
            const int n = __popcll(word & ((1ull << w) - 1));
            if (r >= n) {
                r -= n;
                at += w;
                word >>= w;
            }
        }
        const int part = wave % per_row;
        if (part == 0 && lane == 0) idx_out[p] = at;
        copy_row<CODES>(x + (int64_t)at * d8, out + (int64_t)p * d8, p, d8, part * 64 + lane, per_row * 64, q, tiles);
    }
}

// The rows by themselves, behind a selection that wrote the indices alone.
template <bool CODES>
__global__ __launch_bounds__(256) void gather_rows_kernel(const uint4 *__restrict__ x, const int32_t *__restrict__ idx, int d8,
                                                           uint4 *__restrict__ out, const AgqQuant q, char *__restrict__ tiles) {
    const int p = blockIdx.x;
    copy_row<CODES>(x + (int64_t)idx[p] * d8, out + (int64_t)p * d8, p, d8, threadIdx.x, 256, q, tiles);
}

}  // namespace

int agq_launch_log2_attn(const void *p, int64_t H, int64_t S, int64_t D, int causal, int qmax, const int8_t *vq,
                         int e_v, void *o, void *codes, int32_t *score, void *stream) {
    AttnArgs a;
    a.p = (const uint16_t *)p;
    a.v = vq;
    a.o = (__half *)o;
    a.codes = (uint8_t *)codes;
    a.score = score;
    a.H = (int)H;
    a.S = (int)S;
    a.D = (int)D;
    a.causal = causal;
    a.qmax = qmax;
    a.out_scale = ldexpf(1.0f, e_v - qmax);
    // number of compute units of the current device, asked once per device
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
    const unsigned grid = (unsigned)(((S + kQRows - 1) / kQRows) * H);
    if (D <= 128) {
        if (codes) log2_attn_kernel<1, true><<<grid, 256, 0, st>>>(a);
        else log2_attn_kernel<1, false><<<grid, 256, 0, st>>>(a);
    } else {
        if (codes) log2_attn_kernel<2, true><<<grid, 256, 0, st>>>(a);
        else log2_attn_kernel<2, false><<<grid, 256, 0, st>>>(a);
    }
    return (int)hipGetLastError();
}

int agq_launch_prune(const int32_t *score, int64_t S, int64_t n_keep, const void *x, int64_t d, int32_t *idx,
                     void *x_out, const AgqCodes &codes, void *stream) {
    hipStream_t st = (hipStream_t)stream;
    // Up to 512 tokens eight wavefronts and a row for each workgroup, else sixteen, and so many rows that 256 workgroups or
    // so (one a CU) select: with two to four of them on a CU the selections wait for one another.
    const int waves = S <= 512 ? 8 : 16;
    int rows_per_wg = 1;
    if (S > 512)
        while (rows_per_wg < waves && n_keep > (int64_t)rows_per_wg * 256) rows_per_wg *= 2;
    const unsigned grid = (unsigned)((n_keep + rows_per_wg - 1) / rows_per_wg);
    const AgqQuant q = codes.tiles ? agq_make_quant_signed(codes.bits, codes.e, 0) : AgqQuant{};
    auto launch = [&](unsigned workgroups, auto kernel) {
        kernel<<<workgroups, waves * 64, 0, st>>>(score, (int)S, (int)n_keep, rows_per_wg, (const uint4 *)x, (int)(d / 8), idx, (uint4 *)x_out, q, (char *)codes.tiles);
    };
    // Results that lie over the scores: with every workgroup selecting for itself some would still read scores when others
    // write there, so one workgroup writes the indices and a launch behind it the rows: 2048 tokens, 1024 kept, rows of
    // 5120 9.8 us, 300 tokens, 213 rows of 4096 5.6 (one workgroup for the rows too: 286 and 128).
    auto over_scores = [&](const void *out, int64_t bytes) {
        const uintptr_t o = (uintptr_t)out, s = (uintptr_t)score;
        return o < s + (size_t)S * 4 && s < o + (size_t)bytes;
    };
    if (over_scores(idx, n_keep * 4) || over_scores(x_out, n_keep * d * 2)) {
        if (S <= 512) launch(1, prune_rows_kernel<8, 1, false, false>);
        else if (S <= 2048) launch(1, prune_rows_kernel<16, 2, false, false>);
        else launch(1, prune_rows_kernel<16, 8, false, false>);
        (codes.tiles ? gather_rows_kernel<true> : gather_rows_kernel<false>)<<<(unsigned)n_keep, 256, 0, st>>>(
            (const uint4 *)x, idx, (int)(d / 8), (uint4 *)x_out, q, (char *)codes.tiles);
    } else if (S <= 512) launch(grid, codes.tiles ? prune_rows_kernel<8, 1, true, true> : prune_rows_kernel<8, 1, false, true>);
    else if (S <= 2048) launch(grid, codes.tiles ? prune_rows_kernel<16, 2, true, true> : prune_rows_kernel<16, 2, false, true>);
    else launch(grid, codes.tiles ? prune_rows_kernel<16, 8, true, true> : prune_rows_kernel<16, 8, false, true>);
    return (int)hipGetLastError();
}
