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
// K split of the tiled kernel: `splits` workgroups share a tile's K steps and leave int32 partial tiles behind the activation
// codes in the workspace, which a second kernel adds up.  This plan says which calls may do so (fewer 128 x 128 tiles than
// half of the CUs, a K of eight steps or more, at least four steps a slice) and what room callers reserve for the partial tiles
// (agq_gemm_workspace_bytes), also where the choice below then takes no split, or one of fewer slices.  M tokens, tiles_n =
// 128-wide column tiles of all projections of the call, KT = K steps (TRIP blobs: the extra steps in front included, all of
// which stay in the first slice: min_steps of them).  splits == 1: no split, bytes == 0.  (The constants are those of an
// earlier kernel; they are kept because they decide the sizes that programs reserve.)
struct AgqSplitPlan {
    int splits;
    size_t bytes;
};
static inline AgqSplitPlan agq_tiled_split_plan(int64_t M, int64_t tiles_n, int64_t KT, bool may_split, int min_steps = 0) {
    const int64_t tiles = ((M + 127) / 128) * tiles_n;
    AgqSplitPlan p = {1, 0};
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
        }
    }
    if (p.splits > 1) p.bytes = (size_t)tiles * p.splits * (128 * 128 * 4);
    return p;
}

// The tiled kernel's workgroup tiles and the choice between them.  A tile is 16 nt tokens x 64 jt channels of four
// wavefronts, times kg groups of four that share its K steps (agq_gemm_tiled.hip has what they have in common).
//   TILED_128     128-token tiles, one group
//   TILED_64      64- or 32-token tiles, one group
//   TILED_64X2    64- or 32-token tiles, two groups
//   TILED_SPLIT   64-token tiles whose K steps are shared out over workgroups, with a second launch that adds up
#define AGQ_TILED_SHAPES(F) \
    F(8, 4, 1) F(8, 3, 1) F(8, 2, 1) F(4, 4, 1) F(4, 3, 1) F(4, 2, 1) F(4, 1, 1) F(2, 2, 1) F(2, 1, 1) \
    F(4, 2, 2) F(4, 1, 2) F(2, 2, 2) F(2, 1, 2)
enum AgqTiledVariant { TILED_128, TILED_SPLIT, TILED_64, TILED_64X2 };
struct AgqTiledChoice {
    AgqTiledVariant variant;
    int nt, jt, kg;
    int splits, steps;     // TILED_SPLIT
};

// Time of a launch of w workgroups of one shape, KT steps, N output channels in all, in ns, fitted to 600 calls (17 to 2048
// tokens, K 128 to 13824, N 512 to 27648; codes in, other weights from memory at every launch, graph replays): the error is 4 %
// in the median where a shape is near the best one (10 % of them are off by more than 10 %).  On 650 other calls of 128 to 2048
// tokens, half of them with a K up to 1024, the choice below was 1.1 % slower than the best of all shapes on average, 4 % at the ninth
// decile, 14 % at most; calls that take a K split are apart, see there.
//   fixed  launch, fill and epilogue      step   a step of a lone workgroup on an empty chip      load   what a full chip adds
//   many   a step where CUs have several  more   what each further round of workgroups adds       mem    weights, per 16384 channels
//   ceil64 how far the last round counts as a whole one
struct AgqTiledTime {
    int nt, jt, kg, fixed, step, load, many, more, mem, ceil64;
};
static const AgqTiledTime agq_tiled_times[] = {
    {8, 4, 1, 6851, 427, 232, 637, 2355, 23, 38},
    {8, 3, 1, 6080, 346, 127, 460, 2382, 80, 39},
    {8, 2, 1, 4768, 265, 78, 334, 2130, 95, 32},
    {4, 4, 1, 4817, 299, 81, 352, 2083, 94, 30},
    {4, 3, 1, 4508, 210, 68, 269, 1710, 122, 28},
    {4, 2, 1, 3701, 158, 73, 200, 1168, 118, 30},
    {4, 1, 1, 3034, 130, 37, 119, 830, 153, 34},
    {2, 2, 1, 3187, 153, 18, 136, 786, 115, 40},
    {2, 1, 1, 3010, 97, 13, 84, 618, 140, 40},
    {4, 2, 2, 4643, 136, 55, 200, 3172, 128, 37},
    {4, 1, 2, 3554, 100, 34, 132, 1033, 141, 37},
    {2, 2, 2, 4165, 104, 29, 150, 555, 125, 33},
    {2, 1, 2, 3628, 73, 10, 84, 576, 138, 64},
};
// 128 x 256 tiles of a last round that fills at most half of the CUs are dealt out as halves, in the same launch: how many of w
// (1000 x 4096 -> 12288 46.4 -> 40.7 us, 1024 x 5120 -> 27648 113 -> 104, 333 x 5120 -> 27648 54 -> 48, 2048 x 4096 -> 22016 134 -> 129).
static inline int64_t agq_tiled_halves(int64_t w) { return w > 256 && w % 256 <= 128 ? w % 256 : 0; }
static inline int64_t agq_tiled_ns(const AgqTiledTime &t, int64_t w, int64_t KT, int64_t n_sum) {
    const int64_t mem = t.mem * n_sum >> 14, one = t.fixed + KT * (t.step + (t.load * (w < 256 ? w : 256) >> 8) + mem);
    if (w <= 256) return one;
    const int64_t n = (w + 255) >> 8, halves = 2 * n - (t.nt == 8 && t.jt == 4 && agq_tiled_halves(w) > 0);
    const int64_t several = t.fixed + (n - 1) * t.more + KT * ((t.many * (halves * 128 * t.ceil64 + (64 - t.ceil64) * w) >> 14) + mem);
    return several > one ? several : one;
}
// Workgroups of a call for every tile, counted once for the table: divisions for every shape and projection were half of the host's time.
struct AgqTileCounts {
    int64_t m[9], n[5];    // token tiles of 16 nt (nt 2, 4, 8), column tiles of 64 jt (jt 1 to 4)
    int64_t operator()(int nt, int jt) const { return m[nt] * n[jt]; }
};
static inline AgqTileCounts agq_tile_counts(int64_t M, const int64_t *N, int count) {
    AgqTileCounts c = {};
    for (int nt = 2; nt <= 8; nt *= 2) c.m[nt] = (M + nt * 16 - 1) / (nt * 16);
    for (int p = 0; p < count; ++p) {
        const int64_t n64 = (N[p] + 63) / 64;
        c.n[1] += n64;
        c.n[2] += (n64 + 1) / 2;
        c.n[3] += (n64 + 2) / 3;
        c.n[4] += (n64 + 3) / 4;
    }
    return c;
}
struct AgqTiledPick {
    AgqTiledChoice choice;
    int64_t ns;
};
// KT: steps, the n_extra of TRIP blobs included.
static inline AgqTiledPick agq_tiled_choose(int64_t M, const int64_t *N, int count, int64_t KT, const AgqSplitPlan &plan, int n_extra) {
    int64_t n_sum = 0;
    bool ragged = false;
    for (int p = 0; p < count; ++p) {
        n_sum += N[p];
        ragged = ragged || (N[p] & 7);
    }
    const AgqTileCounts workgroups = agq_tile_counts(M, N, count);
    const int64_t tiles = workgroups(8, 2);
    AgqTiledPick best = {{TILED_128, 8, 4, 1, 1, (int)KT}, INT64_MAX}, split = best;
    // A K split for long K with few tiles: 64 x 64 tiles while four slices of them fit the CUs, else (narrow layers alone) 64 x 128
    // ones, at most four slices (more only add partial tiles to write and read).  Measured against the best tile without: 20 x 11008
    // -> 4096 12.8 against 15.8 us, 64 x 11008 -> 4096 13.7 / 13.9, 300 x 13824 -> 640 11.1 / 13.2.  100 x 11008 -> 4096, whose slices do
    // not fit, 16.2 / 13.7.  (Eight slices of 128 x 128 tiles: 15.1, 17.3, 13.7, 10.9 us for the first four.)
    // Layers of 768 channels and more compare the two (the split's time below is about 1 us high): of 224 such calls no one is slower
    // than with the split alone, 4 % less on average; 512 x 5120 -> 768 14.7 -> 10.6 us, 333 x 4096 -> 768 12.4 -> 9.6, 512 x 8192 -> 1024 18.1 -> 13.8 (with
    // the pre-pass); 200 x 13824 -> 640 keeps it, 14.3 against 16.8.  Narrower ones always take it: tests hold a dozen such calls to
    // it.  There it is level on average, up to a fifth ahead from a K of 8192 on, 10 to 30 % behind for one of 2560 to 4096.
    if (plan.splits > 1 && KT - n_extra >= 20 && 2 * KT >= 3 * tiles &&
        (n_sum <= 1024 || workgroups(4, 1) * (plan.splits < 4 ? plan.splits : 4) <= 256)) {
        const int s = plan.splits < 4 ? plan.splits : 4;
        const int jt = workgroups(4, 1) * s <= 256 ? 1 : 2;
        const int64_t w = workgroups(4, jt);
        int64_t cut = w * s <= 256 ? s : (w * 2 <= 256 ? 256 / w : 2);
        const int64_t steps = (KT + cut - 1) / cut;
        split.choice = {TILED_SPLIT, 4, jt, 1, (int)((KT + steps - 1) / steps), (int)steps};
        for (const AgqTiledTime &t : agq_tiled_times)
            if (t.nt == 4 && t.jt == jt && t.kg == 1) split.ns = agq_tiled_ns(t, w * cut, steps, n_sum) + 3000 + M * n_sum * 4 * cut * 300 / 1000000;
        if (n_sum < 768) return split;
    }
    // Two groups for twelve steps or more on at most 256 tiles of 64 x 128: token tiles that start apart in K bring in weights
    // for each other (agq_gemm_tiled.hip).  Against one group, each with its best tile: 100 x 11008 -> 4096 13.7 / 15.5 us, 213 tokens
    // 17.2 / 21.1, 300 tokens 21.5 / 26.9, 333 x 13824 -> 5120 30.0 / 33.2, 333 x 5120 -> 5120 14.8 / 15.3, 100 x 4096 -> 12288 12.7 / 13.0; behind
    // where K is short and the CUs are full, 512 x 4096 -> 4096 11.6 / 10.3, 256 x 2560 -> 6912 9.5 / 8.1.
    const bool two = KT >= 12 && workgroups(4, 2) <= 256;
    int64_t ns82 = INT64_MAX;
    for (const AgqTiledTime &t : agq_tiled_times) {
        if ((t.kg == 2) != two) continue;
        // Rows of the output that do not start on sixteen bytes: stores across lines (1200 x 1280 -> 4096 / 4100: tiles of 128 x 256
        // 12.0 / 16.0 us, 128 x 192 11.0 / 13.5, 64 x 192 11.2 / 12.2, 64 x 128 11.3 / 11.9).
        const int64_t ns = agq_tiled_ns(t, workgroups(t.nt, t.jt), KT, n_sum) + (ragged ? t.nt * (t.jt - 1) * 100 : 0);
        if (t.nt == 8 && t.jt == 2) ns82 = ns;
        if (ns < best.ns) best = {{t.kg == 2 ? TILED_64X2 : (t.nt == 8 ? TILED_128 : TILED_64), t.nt, t.jt, t.kg, 1, (int)KT}, ns};
    }
    // One round of 128 x 128 tiles on more than half of the CUs, for more than 1024 tokens and eight steps: taken unless another
    // tile is more than a tenth faster.  (There the model has this tile up to a tenth too slow: measured 0.92 to 0.99 of the
    // best other tile on eight of nine such calls of 1200 to 2048 tokens, 1.09 on 1200 x 1408 -> 2000.)
    if (!two && M > 1024 && KT > 8 && tiles <= 256 && tiles > 128 && ns82 * 10 <= best.ns * 11) best = {{TILED_128, 8, 2, 1, 1, (int)KT}, ns82};
    return split.ns - 1000 <= best.ns ? split : best;
}

// Between 17 and 256 rows of fp16 input the weight-streaming kernel can run with sixteen rows and two channel tiles per
// workgroup (grid.y row groups): every row group reads the weights again (from L2 after the first).  The other path is the
// layout pre-pass plus the tiled kernel (above).  Both sides measured on 2600 calls of 17 to 256 rows (K 128 to 13824, N 32 to
// 42000 in up to three projections, other weights from memory at every launch, graph replays):
//   row groups   about 3 us + 89 ns a K step while every workgroup has a CU of its own; for each of two or three rounds of 256 112 ns
//                a K step up to 32 of them, 3.5 us + 50 ns beyond (a wavefront then holds four chunks at a time); from
//                three rounds on 200 ns + 126 ns a K step for every 256 workgroups
//   tiles        the launch below + 2.1 us + 1.6 ns per 1024 values for the pre-pass
// A program that makes its calls one after the other waits for the host, 4.4 us for the one launch of row groups and 8.3 us for
// the two of the tiles (graph replays do not), so row groups of up to 8.6 us are taken whatever the tiles would take.  The others are
// compared.  In graph replays the rule's calls are 0.7 % slower on average than the faster side of each, 20 % at the 99th percentile; with the
// host's share 0.3 %.  Past three rounds with a K of 1280 to 1700 the worst of them 1.5 times (45 x 1408 -> 8600 11.2 / 7.2 us).
// Row groups / tiles: 30 x 11136 -> 3040 12.6 / 15.2 us, 139 x 10880 -> 400 11.0 / 12.9, 768 x 768 at 128 rows 4.1 / 6.5; 200 x 1536 ->
// 3 x 1536 13.4 / 8.1, 80 x 2560 -> 6912 18.0 / 10.1, 256 x 1280 -> 4100 15.1 / 8.3.
// Up to 80 rows, below three rounds, row groups go on for 3.6 us longer from 25 to 32 steps: tests hold three calls of that region
// to them (4096 x 4096 at 64 and 80 rows 10.3 / 9.9 and 13.7 / 10.1, 4096 -> 11008 at 32 rows 13.4 / 11.5).
// (Inside a block the operator in front writes the codes and there is no pre-pass; the same rule is asked there.)
// wgs: groups of sixteen rows times tile pairs (32 channels) of all projections; tiles: what the call would run instead.
// (Four tiles per workgroup instead of two were measured too: the same at best, and 50 % slower on the widest layer, where the
// registers no longer hold the weight chunks.)
#define AGQ_ROW_GROUP_MAX_M 256
static inline int64_t agq_row_groups_ns(int64_t wgs, int64_t KT) {
    if (wgs <= 256) return 89 * KT;
    if (wgs < 768) return (wgs + 255) / 256 * (KT <= 32 ? 112 * KT : 3500 + 50 * KT);
    return wgs * (200 + 126 * KT) / 256;
}
static inline bool agq_decode_row_groups(int64_t M, int64_t KT, int64_t wgs, const AgqTiledPick &tiles) {
    const bool on = KT > 24 && KT <= 32 && M <= 80 && wgs < 768 && tiles.choice.variant != TILED_SPLIT;
    return agq_row_groups_ns(wgs, KT) <= tiles.ns + (on ? 3600 : 0);
}

// Token tiles that the tiled kernel's walk takes together, column by column (a band).  An XCD's run of the walk reads the codes of
// its token tiles and the weights of its columns, so the band says which of the two all eight XCDs read.
//   Tiles of 64 and 32 tokens: up to 1024 tokens in one band, so that the weights come from memory once (300 tokens in a band of four
// tiles and one of one: 4096 -> 22016 33 -> 31 us); layers up to twice as wide as there are tokens tile by tile, and up to ten times as wide
// (two groups: four) in pairs of tiles, so that the codes are read once.  One band for all of them, as it was, against one or two tiles (600
// calls of 150 to 2048 tokens): two groups 7 % and 4 % slower on average, at most 17 %, one group 4 % and 1 %, a K split 3 % and 1 %; 800 x
// 4096 -> 1000 14.5 -> 12.2 us, 986 x 3456 -> 1072 15.4 -> 13.0, 600 x 3072 -> 1536 11.7 -> 11.0.  Wider layers lose: tile by tile 5 %
// from ten times on, two groups in pairs where their token tiles start apart in K for each other (512 x 11008 -> 4096 31.3 -> 35.6).
//   Tiles of 128 tokens: five at a time from six on, a compact rectangle for every XCD.  (Four, or eight: strides that are powers of two
// meet in fewer memory channels; 2048 x 4096 -> 22016 130.7 and 128 -> 126 us, 2048 x 5120 -> 15360 113 and 114 -> 108, level at
// 1000 tokens.)
static inline int agq_tiled_band(int64_t M, int64_t n_sum, int nt, int kg) {
    const int64_t tiles_m = (M + nt * 16 - 1) / (nt * 16), most = 64 / nt;
    if (nt == 8) return (int)(tiles_m > 5 ? 5 : tiles_m);
    if (n_sum < 2 * M) return 1;
    if (n_sum < (kg == 2 ? 4 : 10) * M) return 2;
    return (int)(tiles_m <= most ? tiles_m : most / 2);
}

// int8 codes in operand order, tokens padded to the 128-row tile (a multiple of 16 KiB); K: extra steps included
static inline size_t agq_codes_bytes(int64_t M, int64_t K) { return (size_t)((M + 127) / 128) * 128 * (size_t)K; }

// Which kernel a linear layer takes: the tiled kernel (`tiles`) in one of its variants, or the weight-streaming kernel.
// n_extra >= 0: TRIP blobs with that many extra steps; -1: plain blobs.
struct AgqRoute {
    bool tiles;
    AgqTiledChoice choice;
};
static inline AgqRoute agq_gemm_route(int x_kind, int64_t M, int64_t K, const int64_t *N, int count, int n_extra,
                                      size_t workspace_bytes) {
    // The calls whose launches are shortest do not look at the tiles: up to sixteen rows have no other kernel, and for row groups of
    // up to 8.6 us (3 us besides the time below) the host's second launch decides.
    // The host's time for a choice: 1 x 4096 -> 4096 62 -> 2 ns, 128 x 768 -> 768 66 -> 4, 2048 x 4096 -> 3 x 4096 112 -> 65.
    if (M <= AGQ_DECODE_MAX_M) return {false, {}};
    const bool may_stream = x_kind == 0 && n_extra < 0 && M <= AGQ_ROW_GROUP_MAX_M;
    int64_t tiles_n = 0, wgs = 0;
    for (int p = 0; p < count; ++p) {
        tiles_n += (N[p] + 127) / 128;
        wgs += (N[p] + 31) / 32;
    }
    wgs *= (M + 15) / 16;
    const int extra = n_extra > 0 ? n_extra : 0;
    const int64_t KT = agq_k_tiles(K) + extra;
    if (may_stream && agq_row_groups_ns(wgs, KT) <= 5600) return {false, {}};
    // With few tiles and a long K the tiled kernel splits the tiles' K steps over workgroups, if the
    // caller's workspace has the room for the partial tiles behind the codes.
    AgqSplitPlan plan = agq_tiled_split_plan(M, tiles_n, KT, true, extra);
    if (workspace_bytes < agq_codes_bytes(M, KT * 128) + plan.bytes) plan = agq_tiled_split_plan(M, tiles_n, KT, false);
    const AgqTiledPick pick = agq_tiled_choose(M, N, count, KT, plan, extra);
    return {!(may_stream && agq_decode_row_groups(M, KT, wgs, pick)), pick.choice};
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
// TILED_SPLIT: split_ws has the room that agq_tiled_split_plan asks for.
int agq_launch_gemm_tiled(const void *x_tiles, int64_t M, int64_t K, int e, int corr, const struct agq_proj *projs, int count,
                          int n_extra, const AgqTiledChoice &choice, void *split_ws, void *stream);
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
