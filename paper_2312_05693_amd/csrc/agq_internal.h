// Host-side launcher prototypes; every launcher returns hipError_t as int.
#pragma once
#include <stddef.h>
#include <stdint.h>

// geometry of the packed weight blob (see the packer in agq_quant.hip)
static inline int64_t agq_n_tiles_padded(int64_t N) { return ((N + 255) / 256) * 16; }  // 16-row tiles, padded to 256 rows
static inline int64_t agq_k_tiles(int64_t K) { return K / 128; }
// The blob ends with one int32 per (padded) output channel: the sum of its weights, which the
// asymmetric grid's correction term needs.
static inline size_t agq_blob_nibble_bytes(int64_t N, int64_t K) {
    return (size_t)agq_n_tiles_padded(N) * (size_t)agq_k_tiles(K) * 1024;
}
static inline const int32_t *agq_blob_wsum(const void *packed, int64_t N, int64_t K) {
    return (const int32_t *)((const char *)packed + agq_blob_nibble_bytes(N, K));
}

// ---- TRIP blob (Section 4.4, efficient TRIP matrix multiplication).  The input channels whose
// factor alpha is > 0 are served by E extra 128-wide chunks placed in front of the K/128 main
// chunks of every 16-channel tile (their weights are zero in the main chunks): a chunk holds
// channels of one factor only, chunks are ordered by descending factor.  After the nibbles:
//   int32 wsum[Npad]      sum_k 2^alpha[k] w[n,k]
//   int32 meta[32]        meta[c] = factor of extra chunk c; meta[16 + c] = left shift of the
//                         running accumulator after chunk c (Horner: factor minus the next
//                         chunk's factor, the main chunks counting as factor 0)
//   int32 idx[E * 128]    input channel of every slot of the extra chunks, -1 = unused slot
//   int8  alpha[K]        the factors (read by the packer and by unpack)
#define AGQ_TRIP_MAX_E 16   // == AGQ_TRIP_MAX_EXTRA of the public header
struct AgqTripLayout {
    int64_t KT, KTall, Npad;
    size_t nibble_bytes, wsum_off, meta_off, idx_off, alpha_off, total;
};
static inline AgqTripLayout agq_trip_layout(int64_t N, int64_t K, int E) {
    AgqTripLayout L;
    L.KT = agq_k_tiles(K);
    L.KTall = L.KT + E;
    L.Npad = agq_n_tiles_padded(N) * 16;
    L.nibble_bytes = (size_t)agq_n_tiles_padded(N) * (size_t)L.KTall * 1024;
    L.wsum_off = L.nibble_bytes;
    L.meta_off = L.wsum_off + (size_t)L.Npad * 4;
    L.idx_off = L.meta_off + 32 * 4;
    L.alpha_off = L.idx_off + (size_t)E * 128 * 4;
    L.total = L.alpha_off + (size_t)((K + 15) / 16) * 16;
    return L;
}

// tokens up to which the weight-streaming kernel is used
#define AGQ_DECODE_MAX_M 16
// K split of the tiled kernel.  A K step of a workgroup takes about as long however few workgroups the launch has (the
// plan counts 470 ns: a single wavefront per SIMD cannot cover its own waits): with few 128 x 128 tiles and a long K
// most CUs idle while a few walk K.  Then `splits` workgroups share a tile's K steps (at least four each, at most one
// workgroup per CU in all) and leave int32 partial tiles behind the activation codes in the workspace,
// which a second kernel adds up.  That costs about 2 us for the launch and 0.45 us per MB of partial tiles
// (written, read back); the plan is the split count with the smallest sum under this model (measured on
// MI355X with an earlier schedule of the loop and resident weights).  Its count is the one that agq_tiled_choose below
// weighs against the other variants with the constants of the present loop, and a plan of one slice is never offered there;
// the sizes that callers reserve (agq_gemm_workspace_bytes) hold the plan's partial tiles whether or not the choice then
// takes the split.  M tokens, tiles_n = 128-wide column tiles of all projections of the call, KT = K steps (TRIP
// blobs: the extra steps in front included, all of which stay in the first slice: min_steps of them).
// splits == 1: no split, bytes == 0.
struct AgqSplitPlan {
    int splits, steps;
    size_t bytes;
};
static inline AgqSplitPlan agq_tiled_split_plan(int64_t M, int64_t tiles_n, int64_t KT, bool may_split, int min_steps = 0) {
    const int64_t tiles = ((M + 127) / 128) * tiles_n;
    AgqSplitPlan p = {1, (int)KT, 0};
    if (!may_split || tiles < 1 || tiles * 2 > 256 || KT < 8) return p;
    const int64_t part_bytes = ((M + 31) / 32) * 32 * tiles_n * 512;   // per split: rows that hold tokens x columns x 4
    int64_t least = KT * 470;
    for (int64_t s = 2; s <= KT / 4 && s * tiles <= 256; ++s) {
        const int64_t steps = (KT + s - 1) / s;
        if ((KT + steps - 1) / steps != s || steps < min_steps) continue;   // the same steps with fewer workgroups exist
        const int64_t cost = steps * 470 + 2000 + part_bytes * s * 450 / 1000000;
        if (cost < least) {
            least = cost;
            p.splits = (int)s;
            p.steps = (int)steps;
        }
    }
    if (p.splits > 1) p.bytes = (size_t)tiles * p.splits * (128 * 128 * 4);
    return p;
}

// The tiled kernel's variants and the choice between them: the one with the smallest time under a model of the launch,
// a fixed part and a time per K step that depends on how many workgroups share the chip (KT steps, w workgroups).
//   TILED_128     128-token tiles, at most two workgroups on a CU
//   TILED_SPLIT   the same with the K split above
//   TILED_64      64-token tiles, at most three on a CU: half of the MFMAs per step for two thirds of the operand bytes, so
//                 about 15 % dearer where the chip is full, but finer to deal out
//   TILED_64X2    64-token tiles with the K steps of a tile shared by two groups of four wavefronts of one workgroup: at
//                 most one workgroup per CU, whose two wavefronts per SIMD hide each other's waits
// Measured (us, the GEMM launch alone, other weights from HBM at every launch, as a model's layers have it;
// 128 / split / 64 / 64x2):
//   4096 -> 4096     100 tokens 16.4 / 13.9 / 14.2 / 12.2, 300 tokens 16.7 / - / 14.7 / 12.5, 512 tokens 17.1 / - / 15.4 / 13.9
//   11008 -> 4096    100 tokens 39.3 / 19.7 / 35.1 / 27.3, 213 tokens 39.1 / 23.6 / 35.2 / 27.4, 300 tokens 39.2 / 30.0 / 35.6 / 28.2
//   4096 -> 12288    100 tokens 17.4 / - / 15.6 / 13.7, 213 tokens 19.1 / - / 20.8 / -, 300 tokens 27.9 / - / 23.4 / -
//   4096 -> 22016    100 tokens 20.0 / - / 22.3 / 25.7, 213 tokens 31.3 / - / 33.0 / -, 300 tokens 42.2 / - / 41.5 / -
//   5120 -> 5120     333 tokens 21.5 / - / 19.5 / 16.6, 1024 tokens 35.9 / - / 37.0 / -
//   4096 -> 22016    1000 tokens 89 / - / 101 / -, 2048 tokens 157 / - / 186 / -
// The model is within 10 % of these for 128-token, split and two-group tiles.  For 64-token tiles it is up to 15 % high
// where two or three of them share a CU and 22 % high at 2048 tokens: of the calls above, 4096 -> 22016 at 300 tokens
// goes to 128-token tiles for it, 2 % slower than 64-token ones.
enum AgqTiledVariant { TILED_128, TILED_SPLIT, TILED_64, TILED_64X2 };
struct AgqTiledChoice {
    AgqTiledVariant variant;
    int64_t cost_ns;
};
static inline AgqTiledChoice agq_tiled_choose(int64_t M, int64_t tiles_n, int64_t KT, const AgqSplitPlan &plan, int n_extra = 0) {
    const int64_t w = ((M + 127) / 128) * tiles_n, w64 = ((M + 63) / 64) * tiles_n;
    auto at_least = [](int64_t a, int64_t b) { return a > b ? a : b; };
    const int64_t step = w <= 256 ? 360 + w * 11 / 20 : (w <= 512 ? 700 + (w - 256) * 8 / 5 : at_least(1300, w * 187 / 100));
    AgqTiledChoice c = {TILED_128, 4500 + KT * step};
    auto offer = [&c](AgqTiledVariant v, int64_t cost) {
        if (cost < c.cost_ns) c = {v, cost};
    };
    if (plan.splits > 1) {
        const int64_t part_bytes = ((M + 31) / 32) * 32 * tiles_n * 512;
        offer(TILED_SPLIT, 6500 + plan.steps * (360 + w * plan.splits * 11 / 20) + part_bytes * plan.splits * 450 / 1000000);
    }
    const int64_t step64 = w64 <= 256 ? 300 + w64 * 7 / 20 : (w64 <= 768 ? 460 + (w64 - 256) * 21 / 20 : at_least(1360, w64 * 127 / 100));
    offer(TILED_64, 4000 + KT * step64);
    if (w64 <= 256 && KT > 1) offer(TILED_64X2, 4800 + at_least((KT + 1) / 2, n_extra) * (430 + w64 * 3 / 4));
    return c;
}

// Between 17 and 256 rows of fp16 input the weight-streaming kernel can run with sixteen rows and two channel
// tiles per workgroup (grid.y row groups): every row group reads the weights again (from L2 after the first),
// about 3 us + 0.24 us per MB read in all, more when the workgroups fill the last round of 256 CUs badly.  The
// other path is the layout pre-pass (about 3 us with the gap behind it) plus the tiled kernel (above).  Measured
// (row groups against pre-pass and tiles): 4096 x 4096 at 32 / 64 / 100 rows 6.4 / 11.0 / 18.1 against about 13 us at
// any of them; 768 x 768 at 128 rows 4.1 against 8.2 us.  (The two 3 us cancel in the rule.  Inside a block the operator in
// front writes the codes and there is no pre-pass; the same rule is asked there, so between 17 and about 100 rows a block
// may keep row groups, or tiles, a few rows too long.)  wg_pairs: tile pairs (32 channels) of all projections;
// tiled_ns: the cost of the variant the call would run instead.  (Four tiles per workgroup instead of two were measured
// too: the same at best, and 50 % slower on the widest layer, where the registers no longer hold the weight chunks.)
#define AGQ_ROW_GROUP_MAX_M 256
static inline bool agq_decode_row_groups(int x_kind, int64_t M, int64_t K, int64_t n_sum, int64_t wg_pairs,
                                         int64_t tiled_ns) {
    if (x_kind != 0 || M <= AGQ_DECODE_MAX_M || M > AGQ_ROW_GROUP_MAX_M) return false;
    const int64_t groups = (M + 15) / 16, wgs = groups * wg_pairs;
    int64_t read_ns = groups * (K * n_sum / 2) * 240 / 1000000;
    if (wgs < 768) read_ns = read_ns * ((wgs + 255) / 256 * 256) / wgs;   // a short last round costs a whole one
    return read_ns <= tiled_ns;
}

// int8 codes in operand order, tokens padded to the 128-row tile (a multiple of 16 KiB); K: extra steps included
static inline size_t agq_codes_bytes(int64_t M, int64_t K) { return (size_t)((M + 127) / 128) * 128 * (size_t)K; }

// Which kernel a linear layer takes: the tiled kernel (`tiles`) in one of its variants, or the weight-streaming kernel.
// n_extra >= 0: TRIP blobs with that many extra steps; -1: plain blobs.
struct AgqRoute {
    bool tiles;
    AgqSplitPlan plan;
    AgqTiledChoice choice;
};
static inline AgqRoute agq_gemm_route(int x_kind, int64_t M, int64_t K, const int64_t *N, int count, int n_extra,
                                      size_t workspace_bytes) {
    int64_t tiles_n = 0, wg_pairs = 0, n_sum = 0;
    for (int p = 0; p < count; ++p) {
        tiles_n += (N[p] + 127) / 128;
        wg_pairs += (N[p] + 31) / 32;
        n_sum += N[p];
    }
    // With few tiles and a long K the tiled kernel splits the tiles' K steps over workgroups, if the
    // caller's workspace has the room for the partial tiles behind the codes.
    const int extra = n_extra > 0 ? n_extra : 0;
    const int64_t KT = agq_k_tiles(K) + extra;
    AgqRoute r = {false, agq_tiled_split_plan(M, tiles_n, KT, true, extra), {}};
    if (workspace_bytes < agq_codes_bytes(M, KT * 128) + r.plan.bytes) r.plan = agq_tiled_split_plan(M, tiles_n, KT, false);
    r.choice = agq_tiled_choose(M, tiles_n, KT, r.plan, extra);
    r.tiles = M > AGQ_DECODE_MAX_M && (n_extra >= 0 || !agq_decode_row_groups(x_kind, M, K, n_sum, wg_pairs, r.choice.cost_ns));
    return r;
}

// K steps up to which a launch of five to sixteen rows with several channel tiles per CU takes the K-sliced kernel
#define AGQ_SLICE_MAX_KT 64
// Whether a workgroup of the per-tile kernel serves a pair of channel tiles for five to sixteen rows (fp16 input, plain
// blobs, a K beyond the K-sliced kernel's; more than sixteen rows always run in pairs).  The pair quantizes the activation
// once for both tiles; with 256 CUs its tiles come in `pairs` rounds, single tiles in `ones`.
// From nine rows on a workgroup of single tiles has its CU to itself, so every round saved counts: K = 11008, 16 rows,
// N = 5120 (2 rounds -> 1) 19.1 -> 13.4 us, 9600 (3 -> 2) 28.1 -> 24.6, 16384 (4 -> 2) 39.3 -> 29.0, 16500 (5 -> 3) 45.1 ->
// 36.0; 9 rows 24.8 -> 21.9 at 9600.  With five to eight rows two workgroups of single tiles share a CU, so one round of
// pairs takes as long as two of them: pairs have to halve the rounds (K = 11008, 8 rows, N = 6000 13.6 -> 12.1 us, 16384
// 28.0 -> 25.5, but 9600 19.3 -> 21.6 and 16500 30.2 -> 31.7), and at five and six rows, beyond one round of them, to do so
// with the last two rounds of single tiles nearly full (5 rows, 16384 26.7 -> 25.8, 14000 24.0 -> 24.8).  Where one round
// holds all single tiles the pair leaves half of the CUs idle.
static inline bool agq_decode_pairs(int x_kind, bool trip, int64_t M, int64_t KT, int64_t tiles, int64_t tile_pairs) {
    if (x_kind != 0 || trip || M <= 4 || M > AGQ_DECODE_MAX_M || KT <= AGQ_SLICE_MAX_KT) return false;
    const int64_t ones = (tiles + 255) / 256, pairs = (tile_pairs + 255) / 256;
    if (M > 8) return pairs < ones;
    return 2 * pairs == ones && (pairs == 1 || M > 6 || tiles > ones * 256 - 128);
}

int agq_launch_calibrate(const void *x, int64_t M, int64_t K, int64_t ldx, int bits, int32_t *e_dev, void *stream);
int agq_launch_quantize(const void *x, int64_t M, int64_t K, int64_t ldx, int bits, int e, int zp,
                        void *out, int64_t ld_out_bytes, int out_bits, void *stream);
int agq_launch_prepack_act(const void *x, int x_kind, int bits, int64_t M, int64_t K, int64_t ldx, int e, int zp,
                           void *out, void *stream);
int agq_launch_pack(const int8_t *wq, int64_t N, int64_t K, void *packed, int32_t *bad, void *stream);
int agq_launch_unpack(const void *packed, int64_t N, int64_t K, int8_t *wq, void *stream);
struct agq_proj;
// The linear layer behind every agq_gemm_w4a* call of the public header (argument checks, choice of kernel,
// launches); returns an agq_status.  check_only: the host-side argument checks alone.
int agq_gemm_w4_run(int bits, const void *x, int x_kind, int64_t M, int64_t K, int64_t ldx, int e, int zp,
                    const struct agq_proj *projs, int count, void *workspace, size_t workspace_bytes, void *stream,
                    bool check_only);
// The same in two halves, for a producer that writes the tiled kernel's codes itself (fp16 values through Eq.2, signed
// grid): whether the call would take that kernel, and the call on codes that lie in the workspace already.
bool agq_gemm_takes_tiles(int64_t M, int64_t K, const struct agq_proj *projs, int count, size_t workspace_bytes);
int agq_gemm_w4_tiles(int64_t M, int64_t K, int e, const struct agq_proj *projs, int count, void *workspace,
                      size_t workspace_bytes, void *stream);
// n_extra >= 0 with TRIP blobs (all packed with the same factors, fp16 input); -1 for plain blobs
int agq_launch_gemm_decode(const void *x, int x_kind, int bits, int64_t M, int64_t K, int64_t ldx, int e, int zp,
                           const struct agq_proj *projs, int count, int n_extra, void *stream);
// K counts the main chunks only; with TRIP blobs (all packed with the same factors) x_tiles and the blobs hold
// n_extra more steps in front.  The `count` projections of the activation run as one launch.
// TILED_SPLIT: split_ws has room for the partial tiles that `plan` describes.
int agq_launch_gemm_tiled(const void *x_tiles, int64_t M, int64_t K, int e, int corr, const struct agq_proj *projs, int count,
                          int n_extra, AgqTiledVariant variant, const AgqSplitPlan &plan, void *split_ws, void *stream);
int agq_launch_trip_search(const void *x, int64_t M, int64_t K, int64_t ldx, int bits, int e, int zp, int kmax,
                           int8_t *alpha, void *stream);
int agq_trip_count_extra(const int8_t *alpha_host, int64_t K);   // number of extra chunks, -1 = bad factors or too many
int agq_launch_pack_trip(const int8_t *wq, int64_t N, int64_t K, const int8_t *alpha_host, void *packed, int32_t *bad,
                         void *stream);
int agq_launch_unpack_trip(const void *packed, int64_t N, int64_t K, int n_extra, int8_t *wq, void *stream);
int agq_launch_prepack_trip(const void *x, int bits, int64_t M, int64_t K, int64_t ldx, int e, int zp,
                            const void *packed, int64_t N, int n_extra, void *out, void *stream);
// Eq.2's unsigned grid (zp > 0) inside the GEMMs: codes travel as q - 2^(b-1) (signed, what the
// int8 MFMA takes) and sum_k (q - zp) w = sum_k (q - 2^(b-1)) w + corr * sum_k w.
static inline int agq_zp_corr(int bits, int zp) { return zp ? (1 << (bits - 1)) - zp : 0; }
int agq_launch_log2_attn(const void *p, int64_t H, int64_t S, int64_t D, int causal, int qmax,
                         const int8_t *vq, int e_v, void *o, void *codes, int32_t *score, void *stream);
// codes (optional): where Eq.2's codes of every value go as well, in the operand order of the tiled GEMM
struct AgqCodes {
    void *tiles = nullptr;
    int bits = 8, e = 0;
};
// o_codes and the code map (codes) exclude each other
int agq_launch_qk_log2_attn(const int8_t *q, const int8_t *k, const int8_t *v, int64_t H, int64_t S, int64_t D, int causal,
                            int qmax, int e_q, int e_k, int e_v, void *o, void *codes, int32_t *score, const AgqCodes &o_codes,
                            void *stream);
int agq_launch_prune(const int32_t *score, int64_t S, int64_t n_keep, const void *x, int64_t d,
                     int32_t *idx, void *x_out, const AgqCodes &codes, void *stream);

// ---- fp16 operators of a block (agq_block.hip)
// res != NULL: x1 = fp16(res[idx ? idx[r] : r] + x[r]) is written to x1_out and normalised; pos_out / idx_out
// (optional) receive pos[...] and the source row of every output row
int agq_launch_rmsnorm(const void *x, const void *res, const int32_t *idx, const void *g, void *x1_out, void *y, int64_t rows,
                       int64_t d, double eps, const int32_t *pos, int32_t *pos_out, int32_t *idx_out, const AgqCodes &codes,
                       void *stream);
// q_q != NULL: rotate q and k, Eq.2 on q, k, v, int8 [H,S_pad,D] out (and zero[0..S_pad) = 0 when given);
// q_q == NULL: rotated fp16 q, k to q_rot, k_rot
int agq_launch_rope(const void *q, const void *k, const void *v, int64_t S, int64_t S_pad, int64_t H, int64_t D,
                    const int32_t *pos, const float *cos_t, const float *sin_t, int64_t P, int e_q, int e_k, int e_v,
                    int8_t *q_q, int8_t *k_q, int8_t *v_q, void *q_rot, void *k_rot, int32_t *zero, void *stream);
int agq_launch_swiglu(const void *gate, const void *up, void *out, int64_t n, void *stream);
// the same for rows of F values, with codes
int agq_launch_swiglu_rows(const void *gate, const void *up, void *out, int64_t rows, int64_t F, const AgqCodes &codes, void *stream);
int agq_launch_add(const void *a, const void *b, void *out, int64_t n, void *stream);
int agq_read_i32(const int32_t *dev, int32_t *host, int n, void *stream);
