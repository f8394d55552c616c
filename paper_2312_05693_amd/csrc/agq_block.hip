// The fp16 operators that Section 4.2's pipeline leaves unquantized, for a LLaMA
// block: RMS normalisation (optionally fused with the residual addition and the
// row gather that follows token pruning), the rotary embedding fused with Eq.2 for
// q, k and v, SwiGLU, and the residual addition.  Each takes fp16 tensors and
// returns fp16 (or Eq.2 codes); the arithmetic in between is float64 with one
// rounding to fp16 at the end, so that a result does not depend on the order of a
// reduction or on the exponential's implementation beyond the last bit of a double.
// SwiGLU's float64 exponential, quotient and rounding take longer than its bytes (1024 x 13824: 28 us for 85 MB).  Most values
// do not need them: an fp32 evaluation whose error is known for every fp16 gate tells the fp16 result wherever both ends of its
// interval round to the same one, and only the others, one in several hundred, take the float64 path; the results are float64's in
// every case (17.7 us; 300 x 11008 8.8 -> 6.6).  The others stream their operands once: they are bound by HBM, or by
// latency where rows are few.  (The same for RMSNorm's and the rotary embedding's results, a product and a rounding
// there: 5-20 % slower than float64.)
#include "agq_device.h"
#include "agq_internal.h"

#include <type_traits>

AgqQuant agq_make_quant_signed(int bits, int e, int zp);   // agq_quant.hip

namespace {

// float64 -> fp16, round to nearest even in ONE step.  The hardware converts
// f64 -> f32 and f32 -> f16; rounding twice to nearest can differ from rounding
// once, so the first step is turned into round-to-odd (truncate, then set the last
// bit when anything was cut off), after which the second rounding is exact: 24
// bits keep two more than the 11 of the target.
__device__ __forceinline__ __half f64_to_f16(double d) {
    float f = (float)d;
    const double back = (double)f;
    if (back != d && fabsf(f) <= 3.0e38f) {   // inexact and not overflowed (NaN compares false)
        uint32_t u = __float_as_uint(f);
        if (fabs(back) > fabs(d)) u -= 1;     // nearest went away from zero: step back to the truncation
        f = __uint_as_float(u | 1u);
    }
    return __float2half_rn(f);
}
__device__ __forceinline__ double h2d(uint16_t h) { return (double)__half2float(__ushort_as_half(h)); }
__device__ __forceinline__ uint16_t d2h(double d) { return __half_as_ushort(f64_to_f16(d)); }

struct Half8 {
    uint16_t v[8];
};
static_assert(sizeof(Half8) == 16, "eight fp16 are one 16-byte access");
__device__ __forceinline__ Half8 load8(const void *p) { return __builtin_bit_cast(Half8, *reinterpret_cast<const uint4 *>(p)); }
__device__ __forceinline__ void store8(void *p, const Half8 &h) { *reinterpret_cast<uint4 *>(p) = __builtin_bit_cast(uint4, h); }

// Eight values as the four words of their access; value i by selects (i may differ from lane to lane).
__device__ __forceinline__ uint16_t pick8(const uint4 &v, int i) {
    const uint32_t lo = (i & 2) ? v.y : v.x, hi = (i & 2) ? v.w : v.z;
    return (uint16_t)(((i & 4) ? hi : lo) >> (16 * (i & 1)));
}
__device__ __forceinline__ void put8(uint4 &v, int i, uint16_t h) {
    const uint32_t sh = 16 * (i & 1), keep = 0xFFFF0000u >> sh, bits = (uint32_t)h << sh;
    if ((i >> 1) == 0) v.x = (v.x & keep) | bits;
    if ((i >> 1) == 1) v.y = (v.y & keep) | bits;
    if ((i >> 1) == 2) v.z = (v.z & keep) | bits;
    if ((i >> 1) == 3) v.w = (v.w & keep) | bits;
}

// The results of an operator on eight values as intervals: both ends of each as fp16 in the halves of a word, the larger
// magnitude in the upper half.  Where the ends are the same finite number, that is the result (rounding is monotonic);
// the check costs four instructions a value and one branch.
struct Ends8 {
    uint32_t w[8], differ = 0, largest = 0;
    __device__ __forceinline__ void set(int i, uint32_t ends) {
        w[i] = ends;
        differ |= ends ^ __builtin_amdgcn_alignbit(ends, ends, 16);
        largest = max(largest, ends & 0x7FFFFFFFu);
    }
    __device__ __forceinline__ bool open() const { return differ != 0 || largest >= 0x7C000000u; }
    __device__ __forceinline__ uint32_t open_mask() const {
        uint32_t m = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i)
            m |= (w[i] != __builtin_amdgcn_alignbit(w[i], w[i], 16) || (w[i] & 0x7C00u) == 0x7C00u) ? 1u << i : 0u;
        return m;
    }
    __device__ __forceinline__ uint4 values() const;
};
// p lo and p hi rounded to fp16 once, in the halves of a word (adding -0 keeps the sign of a zero)
__device__ __forceinline__ uint32_t scaled_ends(float p, float lo, float hi) {
    uint32_t d;
    asm("v_fma_mixlo_f16 %0, %1, %2, %3" : "=v"(d) : "v"(p), "v"(lo), "v"(-0.0f));
    asm("v_fma_mixhi_f16 %0, %1, %2, %3" : "+v"(d) : "v"(p), "v"(hi), "v"(-0.0f));
    return d;
}
__device__ __forceinline__ uint4 Ends8::values() const {      // the low halves
    auto low2 = [](uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); };
    return make_uint4(low2(w[0], w[1]), low2(w[2], w[3]), low2(w[4], w[5]), low2(w[6], w[7]));
}

// silu(z) u in eight values, rounded once.  In fp32: e = 2^(-z log2 e) with the exponent in two parts, 1 + e and its
// reciprocal: off by 2^-22.8 at most, measured over all fp16 z against float64 (the instructions' nominal errors alone would
// allow a little more than the interval has, so it is this measurement that holds it, and a test of every gate with
// every mantissa of a factor); the product z u is exact.  With the rounding of an end itself (2^-24) that is 2^-22.3: the
// interval is 2^-22 to either side.
__device__ __forceinline__ uint16_t swiglu1(uint16_t g, uint16_t u) {
    const double z = h2d(g);
    return d2h(z / (1.0 + exp(-z)) * h2d(u));
}
template <bool F32>
__device__ __forceinline__ Half8 swiglu8(const Half8 &g, const Half8 &u) {
    if constexpr (!F32) {
        Half8 o;
#pragma unroll
        for (int i = 0; i < 8; ++i) o.v[i] = swiglu1(g.v[i], u.v[i]);
        return o;
    }
    Ends8 ends;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float z = __half2float(__ushort_as_half(g.v[i])), p = z * __half2float(__ushort_as_half(u.v[i]));
        const float zc = __builtin_amdgcn_fmed3f(z, -64.0f, 64.0f);    // beyond: 1 / (1 + e) is 1, or the result is 0
        const float t = zc * -0x1.715p0f;                              // thirteen bits of log2(e): exact
        const float k = rintf(t);
        const float f = fmaf(zc, -0x1.1d94aep-14f, t - k);             // the rest of log2(e)
        const float e = __builtin_amdgcn_ldexpf(__builtin_amdgcn_exp2f(f), (int)k);
        const float sg = __builtin_amdgcn_rcpf(1.0f + e);
        ends.set(i, scaled_ends(p, sg * (1.0f - 0x1p-22f), sg * (1.0f + 0x1p-22f)));
    }
    uint4 o = ends.values();
    if (ends.open()) {
        const uint4 gw = __builtin_bit_cast(uint4, g), uw = __builtin_bit_cast(uint4, u);
        for (uint32_t open = ends.open_mask(); open; open &= open - 1) {
            const int i = __ffs((int)open) - 1;
            put8(o, i, swiglu1(pick8(gw, i), pick8(uw, i)));
        }
    }
    return __builtin_bit_cast(Half8, o);
}

// a + b of eight values: fp16 addition rounds the exact sum once
__device__ __forceinline__ Half8 add8(const Half8 &a, const Half8 &b) {
    typedef _Float16 h8 __attribute__((ext_vector_type(8)));
    return __builtin_bit_cast(Half8, __builtin_bit_cast(h8, a) + __builtin_bit_cast(h8, b));
}

// Sum over the lanes of a wavefront, uniform, in steps in the data path of the vector ALU: RMSNorm waits for it in every row
// (six steps through LDS instead: 300 rows of 4096 3.84 against 3.57 us, 2048 of 5120 12.7 against 12.3; requesting the
// gains ahead of it takes registers and loses at 1000 rows, 7.7 -> 8.6).
__device__ __forceinline__ double wave_sum(double v) {
    auto step = [&v](auto ctrl_tag, auto rows_tag) {
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, decltype(ctrl_tag)::value, decltype(rows_tag)::value, 0xF, false);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), decltype(ctrl_tag)::value, decltype(rows_tag)::value, 0xF, false);
        v += __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);     // a lane without a source adds 0
    };
    step(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xF>{});   // shifted right by 1, 2, 4, 8 within sixteen lanes
    step(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xF>{});
    step(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xF>{});
    step(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xF>{});
    step(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xA>{});   // lane 15 to the second and fourth sixteen
    step(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xC>{});   // lane 31 to the upper half
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)u, 63), hi = __builtin_amdgcn_readlane((uint32_t)(u >> 32), 63);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

constexpr int kNormThreads = 256;
constexpr int kNormCache = 4;   // rows up to 4 * 256 * 8 = 8192 elements stay in registers between the two passes

// y[r,:] = x1[r,:] * g / sqrt(mean(x1[r,:]^2) + eps), x1 = x (ADD == false) or
// fp16(res[idx[r],:] + x[r,:]) (ADD == true, x1 also written out, with the positions
// of the surviving rows).
// CODES: the Eq.2 codes of y as well, in the operand order of the tiled GEMM (q, tiles).
template <bool ADD, bool CODES>
__global__ __launch_bounds__(kNormThreads) void rmsnorm_kernel(const uint16_t *__restrict__ x, const uint16_t *__restrict__ res,
                                                              const int32_t *__restrict__ idx, const uint16_t *__restrict__ g,
                                                              uint16_t *__restrict__ x1_out, uint16_t *__restrict__ y, int d,
                                                              double eps, const int32_t *__restrict__ pos,
                                                              int32_t *__restrict__ pos_out, int32_t *__restrict__ idx_out,
                                                              const AgqQuant q, char *__restrict__ tiles) {
    const int r = blockIdx.x, tid = threadIdx.x;
    const int src = (ADD && idx) ? idx[r] : r;
    const uint16_t *xr = x + (size_t)r * d;
    const uint16_t *rr = ADD ? res + (size_t)src * d : nullptr;
    if (ADD && tid == 0) {
        if (pos_out) pos_out[r] = pos[src];
        if (idx_out) idx_out[r] = src;
    }
    Half8 cache[kNormCache];
    double ss = 0.0;
    const int nchunk = d >> 3;
#pragma unroll
    for (int it = 0; it < kNormCache; ++it) {
        const int c = tid + it * kNormThreads;
        if (c < nchunk) {
            Half8 h = load8(xr + c * 8);
            if (ADD) {
                h = add8(load8(rr + c * 8), h);
                store8(x1_out + (size_t)r * d + c * 8, h);
            }
            cache[it] = h;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const double v = h2d(h.v[i]);
                ss += v * v;
            }
        }
    }
    for (int c = tid + kNormCache * kNormThreads; c < nchunk; c += kNormThreads) {   // rows wider than the cache
        Half8 h = load8(xr + c * 8);
        if (ADD) {
            h = add8(load8(rr + c * 8), h);
            store8(x1_out + (size_t)r * d + c * 8, h);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const double v = h2d(h.v[i]);
            ss += v * v;
        }
    }
    ss = wave_sum(ss);
    __shared__ double part[kNormThreads / 64];
    if ((tid & 63) == 0) part[tid >> 6] = ss;
    __syncthreads();
    double tot = 0.0;
#pragma unroll
    for (int w = 0; w < kNormThreads / 64; ++w) tot += part[w];
    const double inv = 1.0 / sqrt(tot / (double)d + eps);
    const uint16_t *src1 = ADD ? x1_out + (size_t)r * d : xr;   // this thread re-reads only what it wrote itself
#pragma unroll
    for (int it = 0; it < kNormCache; ++it) {
        const int c = tid + it * kNormThreads;
        if (c < nchunk) {
            const Half8 gg = load8(g + c * 8);
            Half8 o;
#pragma unroll
            for (int i = 0; i < 8; ++i) o.v[i] = d2h((h2d(cache[it].v[i]) * h2d(gg.v[i])) * inv);
            store8(y + (size_t)r * d + c * 8, o);
            if (CODES)
                *reinterpret_cast<uint2 *>(tiles + agq_code_offset(r, c, d >> 7)) = agq_quant8<true>(__builtin_bit_cast(uint4, o), q);
        }
    }
    for (int c = tid + kNormCache * kNormThreads; c < nchunk; c += kNormThreads) {
        const Half8 h = load8(src1 + c * 8), gg = load8(g + c * 8);
        Half8 o;
#pragma unroll
        for (int i = 0; i < 8; ++i) o.v[i] = d2h((h2d(h.v[i]) * h2d(gg.v[i])) * inv);
        store8(y + (size_t)r * d + c * 8, o);
        if (CODES)
            *reinterpret_cast<uint2 *>(tiles + agq_code_offset(r, c, d >> 7)) = agq_quant8<true>(__builtin_bit_cast(uint4, o), q);
    }
}

// Eq.2 on one fp16 value, signed 8-bit grid, step 2^e (inv = 2^-e): the product is
// exact in fp32, the rounding is to nearest even.
__device__ __forceinline__ uint32_t quant8_1(uint16_t h, float inv) {
    const float r = rintf(__half2float(__ushort_as_half(h)) * inv);
    return (uint32_t)(int)fminf(fmaxf(r, -128.0f), 127.0f) & 0xFFu;
}
__device__ __forceinline__ uint2 quant8_8(const Half8 &h, float inv) {
    uint2 o;
    o.x = quant8_1(h.v[0], inv) | (quant8_1(h.v[1], inv) << 8) | (quant8_1(h.v[2], inv) << 16) | (quant8_1(h.v[3], inv) << 24);
    o.y = quant8_1(h.v[4], inv) | (quant8_1(h.v[5], inv) << 8) | (quant8_1(h.v[6], inv) << 16) | (quant8_1(h.v[7], inv) << 24);
    return o;
}

struct RopeArgs {
    const uint16_t *src[3];   // q, k, v: fp16 [S, H*D]
    int8_t *dst_q[3];         // int8 [H, S_pad, D]            (QUANT)
    uint16_t *dst_h[2];       // rotated q, k: fp16 [S, H*D]   (!QUANT)
    float inv[3];             // 2^-e of q, k, v
    const int32_t *pos;
    const float *cos_t, *sin_t;   // float32 [P, D/2]
    int S, S_pad, H, D, P;
    int32_t *zero;            // optional int32 [S_pad] cleared on the way (the importance score accumulates)
};

// blockIdx.x = token row (0 .. S_pad-1), blockIdx.y = tensor (0 q, 1 k, 2 v).  A work
// item is eight pairs (i, i + D/2) of one head: two 16-byte loads, rotation by the
// angles of (pos[row], i) for q and k, then either Eq.2 and the head-major int8 store
// or the rotated fp16 values (the calibration pass needs those).
template <bool QUANT>
__global__ __launch_bounds__(256) void rope_kernel(const RopeArgs a) {
    const int row = blockIdx.x, t = blockIdx.y;
    const int D = a.D, Dh = D >> 1, per_head = D >> 4;
    const int items = a.H * per_head;
    const bool pad = row >= a.S;
    if (QUANT && a.zero && t == 0 && threadIdx.x == 0) a.zero[row] = 0;
    const int p = pad ? 0 : min(max(a.pos[row], 0), a.P - 1);   // a position outside the table is clamped into it
    // selects instead of indexing with t: the argument record stays in scalar registers
    const uint16_t *src = (t == 0 ? a.src[0] : t == 1 ? a.src[1] : a.src[2]) + (size_t)row * a.H * D;
    const float inv = t == 0 ? a.inv[0] : t == 1 ? a.inv[1] : a.inv[2];
    for (int it = threadIdx.x; it < items; it += 256) {
        const int head = it / per_head, j = (it - head * per_head) * 8;
        uint2 qlo = make_uint2(0u, 0u), qhi = make_uint2(0u, 0u);
        if (!pad) {
            Half8 lo = load8(src + head * D + j), hi = load8(src + head * D + Dh + j);
            if (t < 2) {
                const float4 c0 = *reinterpret_cast<const float4 *>(a.cos_t + (size_t)p * Dh + j);
                const float4 c1 = *reinterpret_cast<const float4 *>(a.cos_t + (size_t)p * Dh + j + 4);
                const float4 s0 = *reinterpret_cast<const float4 *>(a.sin_t + (size_t)p * Dh + j);
                const float4 s1 = *reinterpret_cast<const float4 *>(a.sin_t + (size_t)p * Dh + j + 4);
                const float cs[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
                const float sn[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const double l = h2d(lo.v[i]), h = h2d(hi.v[i]), c = (double)cs[i], s = (double)sn[i];
                    lo.v[i] = d2h(l * c - h * s);
                    hi.v[i] = d2h(h * c + l * s);
                }
            }
            if (!QUANT) {
                if (t < 2) {
                    uint16_t *dh = (t == 0 ? a.dst_h[0] : a.dst_h[1]) + (size_t)row * a.H * D + head * D;
                    store8(dh + j, lo);
                    store8(dh + Dh + j, hi);
                }
                continue;
            }
            qlo = quant8_8(lo, inv);
            qhi = quant8_8(hi, inv);
        }
        if (QUANT) {
            int8_t *dst = (t == 0 ? a.dst_q[0] : t == 1 ? a.dst_q[1] : a.dst_q[2]) + ((size_t)head * a.S_pad + row) * D;
            *reinterpret_cast<uint2 *>(dst + j) = qlo;
            *reinterpret_cast<uint2 *>(dst + Dh + j) = qhi;
        }
    }
}

// From how many values on SwiGLU evaluates in fp32 first.  With fewer there is at most one workgroup on a CU, whose
// latency the float64 path behind the fp32 one lengthens: 8192 to 400000 values 0.2-0.35 us slower, 600000 and 800000 0.06
// faster, 1.2 million 4.5 -> 4.1 us, 2.5 million 6.8 -> 5.5.
constexpr int64_t kSwigluF32 = 256 * 256 * 8;

// a = silu(gate) * up, eight values per thread
template <bool F32>
__global__ __launch_bounds__(256) void swiglu_kernel(const uint16_t *__restrict__ gate, const uint16_t *__restrict__ up,
                                                     uint16_t *__restrict__ out, size_t nchunk) {
    const size_t c = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (c >= nchunk) return;
    store8(out + c * 8, swiglu8<F32>(load8(gate + c * 8), load8(up + c * 8)));
}

// the same over rows of F8 chunks (grid: chunks of a row, rows), with the rows' Eq.2 codes in the operand order of the
// tiled GEMM
template <bool F32>
__global__ __launch_bounds__(256) void swiglu_codes_kernel(const uint16_t *__restrict__ gate, const uint16_t *__restrict__ up,
                                                           uint16_t *__restrict__ out, int F8, const AgqQuant q,
                                                           char *__restrict__ tiles) {
    const int c = blockIdx.x * 256 + threadIdx.x, r = blockIdx.y;
    if (c >= F8) return;
    const size_t at = ((size_t)r * F8 + c) * 8;
    const Half8 o = swiglu8<F32>(load8(gate + at), load8(up + at));
    store8(out + at, o);
    *reinterpret_cast<uint2 *>(tiles + agq_code_offset(r, c, F8 >> 4)) = agq_quant8<true>(__builtin_bit_cast(uint4, o), q);
}

__global__ __launch_bounds__(256) void add_kernel(const uint16_t *__restrict__ a, const uint16_t *__restrict__ b,
                                                  uint16_t *__restrict__ out, size_t nchunk) {
    const size_t c = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (c >= nchunk) return;
    store8(out + c * 8, add8(load8(a + c * 8), load8(b + c * 8)));
}

}  // namespace

int agq_launch_rmsnorm(const void *x, const void *res, const int32_t *idx, const void *g, void *x1_out, void *y, int64_t rows,
                       int64_t d, double eps, const int32_t *pos, int32_t *pos_out, int32_t *idx_out, const AgqCodes &codes,
                       void *stream) {
    if (rows == 0) return 0;
    hipStream_t st = (hipStream_t)stream;
    const AgqQuant q = codes.tiles ? agq_make_quant_signed(codes.bits, codes.e, 0) : AgqQuant{};
    const auto kernel = res ? (codes.tiles ? rmsnorm_kernel<true, true> : rmsnorm_kernel<true, false>)
                            : (codes.tiles ? rmsnorm_kernel<false, true> : rmsnorm_kernel<false, false>);
    kernel<<<(unsigned)rows, kNormThreads, 0, st>>>((const uint16_t *)x, (const uint16_t *)res, idx, (const uint16_t *)g,
                                                    (uint16_t *)x1_out, (uint16_t *)y, (int)d, eps, pos, pos_out, idx_out, q,
                                                    (char *)codes.tiles);
    return (int)hipGetLastError();
}

int agq_launch_rope(const void *q, const void *k, const void *v, int64_t S, int64_t S_pad, int64_t H, int64_t D,
                    const int32_t *pos, const float *cos_t, const float *sin_t, int64_t P, int e_q, int e_k, int e_v,
                    int8_t *q_q, int8_t *k_q, int8_t *v_q, void *q_rot, void *k_rot, int32_t *zero, void *stream) {
    if (q_q ? S_pad == 0 : S == 0) return 0;   // with S == 0 the padding rows are still cleared
    RopeArgs a;
    a.src[0] = (const uint16_t *)q; a.src[1] = (const uint16_t *)k; a.src[2] = (const uint16_t *)v;
    a.dst_q[0] = q_q; a.dst_q[1] = k_q; a.dst_q[2] = v_q;
    a.dst_h[0] = (uint16_t *)q_rot; a.dst_h[1] = (uint16_t *)k_rot;
    a.inv[0] = ldexpf(1.0f, -e_q); a.inv[1] = ldexpf(1.0f, -e_k); a.inv[2] = ldexpf(1.0f, -e_v);
    a.pos = pos; a.cos_t = cos_t; a.sin_t = sin_t;
    a.S = (int)S; a.S_pad = (int)S_pad; a.H = (int)H; a.D = (int)D; a.P = (int)P;
    a.zero = zero;
    hipStream_t st = (hipStream_t)stream;
    if (q_q)
        rope_kernel<true><<<dim3((unsigned)S_pad, 3), 256, 0, st>>>(a);
    else
        rope_kernel<false><<<dim3((unsigned)S, 2), 256, 0, st>>>(a);
    return (int)hipGetLastError();
}

int agq_launch_swiglu(const void *gate, const void *up, void *out, int64_t n, void *stream) {
    if (n == 0) return 0;
    const size_t nchunk = (size_t)n / 8;
    (n >= kSwigluF32 ? swiglu_kernel<true> : swiglu_kernel<false>)<<<(unsigned)((nchunk + 255) / 256), 256, 0, (hipStream_t)stream>>>((const uint16_t *)gate, (const uint16_t *)up,
                                                                                   (uint16_t *)out, nchunk);
    return (int)hipGetLastError();
}

int agq_launch_swiglu_rows(const void *gate, const void *up, void *out, int64_t rows, int64_t F, const AgqCodes &codes, void *stream) {
    const int F8 = (int)(F / 8);
    (rows * F >= kSwigluF32 ? swiglu_codes_kernel<true> : swiglu_codes_kernel<false>)<<<dim3((unsigned)((F8 + 255) / 256), (unsigned)rows), 256, 0, (hipStream_t)stream>>>(
        (const uint16_t *)gate, (const uint16_t *)up, (uint16_t *)out, F8, agq_make_quant_signed(codes.bits, codes.e, 0),
        (char *)codes.tiles);
    return (int)hipGetLastError();
}

int agq_launch_add(const void *a, const void *b, void *out, int64_t n, void *stream) {
    if (n == 0) return 0;
    const size_t nchunk = (size_t)n / 8;
    add_kernel<<<(unsigned)((nchunk + 255) / 256), 256, 0, (hipStream_t)stream>>>((const uint16_t *)a, (const uint16_t *)b,
                                                                                (uint16_t *)out, nchunk);
    return (int)hipGetLastError();
}

// blocking read of a few device words (calibration only)
int agq_read_i32(const int32_t *dev, int32_t *host, int n, void *stream) {
    hipError_t e = hipMemcpyAsync(host, dev, (size_t)n * sizeof(int32_t), hipMemcpyDeviceToHost, (hipStream_t)stream);
    if (e != hipSuccess) return (int)e;
    return (int)hipStreamSynchronize((hipStream_t)stream);
}
