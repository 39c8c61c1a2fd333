// Row-wise kernels around the GEMM: the per-token activation quantiser, the
// offline per-channel weight quantiser + packer, the SiLU*up glue, and the
// glue fused with the quantiser that follows it.  All are one pass over HBM;
// a workgroup owns one row.
#include "common.hpp"
#include "kernels.hpp"

namespace w4a8 {

namespace {

constexpr int kRowThreads = 256;
constexpr int kCache = 8;  // 16-byte chunks a thread keeps in registers between the two passes (K <= 16384)
constexpr int kFewRows = 128;  // token counts up to which the activation quantiser spreads a row over 1024 threads
constexpr int kSomeRows = 256;  // ... and over 512 threads (measured: 3-5 % faster than 256 threads up to 256 rows, 5 % slower at 512)

// maximum over the workgroup; every thread gets the result.  NONNEG: the values are absolute values (the wave's step
// then runs in the vector ALU instead of through six shuffles)
template <int THREADS = kRowThreads, bool NONNEG = false>
__device__ __forceinline__ float block_max(float v, float *scratch) {
    if constexpr (NONNEG) {
        v = wave_max_nonneg(v);
    } else {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
    }
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) scratch[wave] = v;
    __syncthreads();
    float m = scratch[0];
#pragma unroll
    for (int w = 1; w < THREADS / 64; ++w) m = fmaxf(m, scratch[w]);
    return m;
}

// A row's chunks of 16 bytes as a buffer: a chunk past its end reads as zeros and touches no memory, so that a thread's loads stand
// in a row with no branch between them, all in flight at once.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_buffer(const void *row, int chunks) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(row), 0, chunks * 16, 0x00020000);
}
__device__ __forceinline__ v4u row_chunk(__amdgpu_buffer_rsrc_t row, int c) { return __builtin_amdgcn_raw_buffer_load_b128(row, c * 16, 0, 0); }

// fp16( silu(gate) * up ) for eight gate / up pairs, fp32 arithmetic, as four words of two fp16 each.
// silu(g) = g / (1 + e^-g) with the hardware's exp2 and reciprocal (about 1 ulp of fp32 each): the result carries a
// few ulps of fp32 error, three orders of magnitude below the fp16 rounding that follows, and the kernel stays
// bandwidth-bound (the correctly rounded library exp and division cost some 35 vector operations per element and made
// it compute-bound).  exp2 overflows to +inf for very negative g, the reciprocal of that is 0: silu(-65504) = -0.
__device__ __forceinline__ v4u silu_mul8(v4u gv, v4u uv) {
    v4u o;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float y[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const float gt = e ? hi_half(gv[j]) : lo_half(gv[j]);
            const float up = e ? hi_half(uv[j]) : lo_half(uv[j]);
            y[e] = silu_mul_f32(gt, up);
        }
        o[j] = pack_f16x2(y[0], y[1]);
    }
    return o;
}

}  // namespace

// Per-token symmetric int8 quantisation (Sec. 3 "per token"; Eq. (2), z = 0).
// Rows of x are ldx elements apart (ldx = K for a dense matrix; more when x is a column slice of a wider one).
// Loads and stores carry the non-temporal hint: a row is read once and its codes are written once (measured at
// M = 1024 .. 2048, K = 5120: 8 to 11 % off the kernel's time, nothing lost at small M; the GEMM that reads the codes
// next is not slowed).  A row per wave or per two waves, several rows to a workgroup, was slower at every M tried.
// THREADS, CACHE: threads per row and chunks a thread keeps between the passes.  256 x 8 where the rows fill the chip;
// for a few rows (token generation) 1024 x 2, which shortens each thread's share of the one row its compute unit has;
// 512 x 4 in between.
template <int THREADS, int CACHE>
__global__ __launch_bounds__(THREADS, THREADS <= 256 ? 8 : 1) void quantize_act_kernel(const uint16_t *__restrict__ x, int8_t *__restrict__ xq,
                                                              float *__restrict__ s_a, int K, long long ldx) {
    constexpr int kRowThreads = THREADS, kCache = CACHE;  // shadow the file-scope defaults
    __shared__ float scratch[kRowThreads / 64];
    const int m = blockIdx.x;
    const int chunks = K >> 3;  // 8 fp16 = 16 bytes
    const v4u *src = (const v4u *)(x + (size_t)m * (size_t)ldx);

    v4u cache[kCache];
    unsigned amax2 = 0u;
#pragma unroll
    for (int i = 0; i < kCache; ++i) {
        const int c = threadIdx.x + i * kRowThreads;
        cache[i] = v4u{0, 0, 0, 0};
        if (c < chunks) cache[i] = __builtin_nontemporal_load(src + c);
        amax2 = absmax8_packed(cache[i], amax2);
    }
    for (int c = threadIdx.x + kCache * kRowThreads; c < chunks; c += kRowThreads) amax2 = absmax8_packed(src[c], amax2);
    float amax = block_max<kRowThreads, true>(absmax_packed_value(amax2), scratch);

    const RowQuantizer rq(amax, 127.0f, -127.f, 127.f);
    if (threadIdx.x == 0) s_a[m] = rq.scale;  // amax == 0 gives scale 0
    const bool zero_row = amax == 0.f;

    v2u *dst = (v2u *)(xq + (size_t)m * K);
    auto emit = [&](int c, v4u v) {
        v2u o = v2u{0, 0};
        if (!zero_row) {
            float xf[8];
            halves8(v, xf);
            o = rq.packed8_own_max<true>(xf);
        }
        __builtin_nontemporal_store(o, dst + c);
    };
#pragma unroll
    for (int i = 0; i < kCache; ++i) {
        const int c = threadIdx.x + i * kRowThreads;
        if (c < chunks) emit(c, cache[i]);
    }
    for (int c = threadIdx.x + kCache * kRowThreads; c < chunks; c += kRowThreads) emit(c, src[c]);
}

// Eight int4 codes from two words of int8 codes: code j in nibble j (App. A.1, low nibble = even k).
__device__ __forceinline__ unsigned nibbles8(v2u codes) {
    const unsigned lo = codes.x & 0x0F0F0F0Fu, hi = codes.y & 0x0F0F0F0Fu;
    return __builtin_amdgcn_perm(hi | (hi >> 4), lo | (lo >> 4), 0x06040200u);
}

// Per-output-channel symmetric int4 round-to-nearest (Eq. (8),(9), 4 bits, gamma = beta = 1)
// followed by the nibble packing of App. A.1 (low nibble = even k).
// What bounds it: the read of the fp16 rows.  A row is read once, into registers, and the codes take some six vector
// operations per element (codes8, with its clamps and conversions, takes a dozen, as many microseconds as the memory
// does).  Measured, cold rows, N = 27648, K = 5120: 57 us = 6.2 TB/s, against 98 with the row read twice and codes8;
// N = 32768, K = 8192: 165 -> 102 us; N = 12288, K = 4096: 36 -> 23.  THREADS: 128 with short rows, where a thread of
// 256 would hold fewer than three chunks (27648 x 5120: 57 us against 65); 256 with longer ones (5000 x 6944: 18.1 against
// 19.6).  Loads carry the non-temporal hint, the stores do not: the codes are read next, by the kernel that tiles them
// (without the hint on the loads 65 us; with it on the stores 62).
constexpr int kShortRow = 6144;

template <int THREADS, int CACHE>
__global__ __launch_bounds__(THREADS, 8) void quantize_weights_kernel(const uint16_t *__restrict__ w, uint8_t *__restrict__ wp,
                                                                   float *__restrict__ s_w, int K) {
    // The row's maximum is put together from kParts maxima, part w of the chunks c with (c / 64) % kParts = w, for either
    // THREADS: which parts hold a NaN decides what becomes of such a row (fmaxf passes over a part that is NaN), and that
    // does not depend on the launch shape.
    constexpr int kParts = kRowThreads / 64, kOwnParts = kRowThreads / THREADS;
    static_assert(THREADS == kRowThreads || CACHE * THREADS * 8 >= kShortRow, "short rows are held in registers whole");
    __shared__ float scratch[kParts];
    const int n = blockIdx.x;
    const int chunks = K >> 3;
    const v4u *src = (const v4u *)(w + (size_t)n * K);

    v4u cache[CACHE];
    unsigned amax2[kOwnParts] = {};
#pragma unroll
    for (int i = 0; i < CACHE; ++i) {
        const int c = threadIdx.x + i * THREADS;
        cache[i] = v4u{0, 0, 0, 0};
        if (c < chunks) cache[i] = __builtin_nontemporal_load(src + c);
    }
#pragma unroll
    for (int i = 0; i < CACHE; ++i) amax2[i % kOwnParts] = absmax8_packed(cache[i], amax2[i % kOwnParts]);
    if (THREADS == kRowThreads)
        for (int c = threadIdx.x + CACHE * THREADS; c < chunks; c += THREADS) amax2[0] = absmax8_packed(src[c], amax2[0]);
#pragma unroll
    for (int j = 0; j < kOwnParts; ++j) {
        const float part = wave_max_nonneg(absmax_packed_value(amax2[j]));
        if ((threadIdx.x & 63) == 0) scratch[j * (THREADS / 64) + (threadIdx.x >> 6)] = part;
    }
    __syncthreads();
    float amax = scratch[0];
    bool finite_row = scratch[0] < INFINITY;  // false for NaN as well
#pragma unroll
    for (int w = 1; w < kParts; ++w) {
        amax = fmaxf(amax, scratch[w]);
        finite_row &= scratch[w] < INFINITY;
    }

    const RowQuantizer rq(amax, 7.0f, -8.f, 7.f);
    if (threadIdx.x == 0) s_w[n] = rq.scale;
    const bool zero_row = amax == 0.f;

    unsigned *dst = (unsigned *)(wp + (size_t)n * (K >> 1));
    auto emit = [&](int c, v4u v) {
        unsigned o = 0;
        float xf[8];
        halves8(v, xf);
        if (!finite_row && !zero_row) {
            int q[8];
            rq.codes8(xf, q);
#pragma unroll
            for (int j = 0; j < 4; ++j) o |= (unsigned)((q[2 * j] & 15) | ((q[2 * j + 1] & 15) << 4)) << (8 * j);
        } else if (!zero_row) {
            o = nibbles8(rq.packed8_own_max<false>(xf));
        }
        dst[c] = o;
    };
#pragma unroll
    for (int i = 0; i < CACHE; ++i) {
        const int c = threadIdx.x + i * THREADS;
        if (c < chunks) emit(c, cache[i]);
    }
    if (THREADS == kRowThreads)
        for (int c = threadIdx.x + CACHE * THREADS; c < chunks; c += THREADS) emit(c, src[c]);
}

// The same with the clipping strengths of Eq. (9) per output channel: S = max(|gamma max(W)|, |beta min(W)|) / 7.
// Values outside the clipped range saturate at -8 / 7 (Eq. (8)).  gamma / beta may be NULL (= 1).
__global__ __launch_bounds__(kRowThreads, 8) void quantize_weights_clip_kernel(const uint16_t *__restrict__ w,
                                                                            const float *__restrict__ gamma,
                                                                            const float *__restrict__ beta,
                                                                            uint8_t *__restrict__ wp, float *__restrict__ s_w,
                                                                            int K) {
    __shared__ float scratch_hi[kRowThreads / 64];
    __shared__ float scratch_lo[kRowThreads / 64];
    const int n = blockIdx.x;
    const int chunks = K >> 3;
    const v4u *src = (const v4u *)(w + (size_t)n * K);

    float hi = -INFINITY, neg_lo = -INFINITY;  // max(W) and max(-W) = -min(W)
    for (int c = threadIdx.x; c < chunks; c += kRowThreads) {
        float xf[8];
        halves8(src[c], xf);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            hi = fmaxf(hi, xf[j]);
            neg_lo = fmaxf(neg_lo, -xf[j]);
        }
    }
    hi = block_max(hi, scratch_hi);
    neg_lo = block_max(neg_lo, scratch_lo);
    const float g = gamma ? gamma[n] : 1.0f, b = beta ? beta[n] : 1.0f;
    const float top = fmaxf(fabsf(g * hi), fabsf(b * -neg_lo));

    const RowQuantizer rq(top, 7.0f, -8.f, 7.f);
    if (threadIdx.x == 0) s_w[n] = rq.scale;
    const bool zero_row = top == 0.f;

    unsigned *dst = (unsigned *)(wp + (size_t)n * (K >> 1));
    for (int c = threadIdx.x; c < chunks; c += kRowThreads) {
        unsigned o = 0;
        if (!zero_row) {
            float xf[8];
            int q[8];
            halves8(src[c], xf);
            rq.codes8(xf, q);
#pragma unroll
            for (int j = 0; j < 4; ++j) o |= (unsigned)((q[2 * j] & 15) | ((q[2 * j + 1] & 15) << 4)) << (8 * j);
        }
        dst[c] = o;
    }
}

// h = fp16( silu(gate) * up ), gate = columns [0,I), up = columns [I,2I) of a row of gate_up.
__global__ __launch_bounds__(kRowThreads) void silu_mul_kernel(const uint16_t *__restrict__ gate_up, uint16_t *__restrict__ h,
                                                               int I) {
    const int m = blockIdx.y;
    const int c = blockIdx.x * kRowThreads + threadIdx.x;  // 8 outputs per thread
    if (c >= (I >> 3)) return;
    const v4u gv = *((const v4u *)(gate_up + (size_t)m * 2 * I) + c);
    const v4u uv = *((const v4u *)(gate_up + (size_t)m * 2 * I + I) + c);
    *((v4u *)(h + (size_t)m * I) + c) = silu_mul8(gv, uv);
}

// The glue and the quantiser behind it in one pass: h = fp16(silu(gate) * up) is formed in registers (the same
// arithmetic as silu_mul_kernel, so the same fp16 bits), then quantised per token exactly as quantize_act_kernel
// would quantise it.  The fp16 intermediate never goes to memory.  A row is spread over 1024 threads so that a
// thread holds at most two chunks of h (I <= 16384); longer rows recompute h in the second pass.  (Measured at
// M = 1024, I = 13824, cold input: 512 threads with four chunks each, two workgroups per compute unit, are 4 % slower;
// both chunks asked for ahead of the arithmetic 5 % faster beyond 512 rows, 2 to 4 % slower up to there, where this kernel is used;
// non-temporal loads and stores change nothing, in isolation or inside the layer's step.)
constexpr int kFusedThreads = 1024;
constexpr int kFusedCache = 2;

__global__ __launch_bounds__(kFusedThreads) void silu_mul_quantize_kernel(const uint16_t *__restrict__ gate_up,
                                                                          int8_t *__restrict__ xq, float *__restrict__ s_a,
                                                                          int I) {
    __shared__ float scratch[kFusedThreads / 64];
    const int m = blockIdx.x;
    const int chunks = I >> 3;
    const v4u *gate = (const v4u *)(gate_up + (size_t)m * 2 * I);
    const v4u *up = (const v4u *)(gate_up + (size_t)m * 2 * I + I);

    v4u cache[kFusedCache];
    unsigned amax2 = 0u;
#pragma unroll
    for (int i = 0; i < kFusedCache; ++i) {
        const int c = threadIdx.x + i * kFusedThreads;
        cache[i] = v4u{0, 0, 0, 0};
        if (c < chunks) cache[i] = silu_mul8(gate[c], up[c]);
        amax2 = absmax8_packed(cache[i], amax2);
    }
    for (int c = threadIdx.x + kFusedCache * kFusedThreads; c < chunks; c += kFusedThreads)
        amax2 = absmax8_packed(silu_mul8(gate[c], up[c]), amax2);
    const float amax = block_max<kFusedThreads, true>(absmax_packed_value(amax2), scratch);

    const RowQuantizer rq(amax, 127.0f, -127.f, 127.f);
    if (threadIdx.x == 0) s_a[m] = rq.scale;
    const bool zero_row = amax == 0.f;

    v2u *dst = (v2u *)(xq + (size_t)m * I);
    auto emit = [&](int c, v4u v) {
        v2u o = v2u{0, 0};
        if (!zero_row) {
            float xf[8];
            halves8(v, xf);
            o = rq.packed8_own_max<true>(xf);
        }
        dst[c] = o;
    };
#pragma unroll
    for (int i = 0; i < kFusedCache; ++i) {
        const int c = threadIdx.x + i * kFusedThreads;
        if (c < chunks) emit(c, cache[i]);
    }
    for (int c = threadIdx.x + kFusedCache * kFusedThreads; c < chunks; c += kFusedThreads)
        emit(c, silu_mul8(gate[c], up[c]));
}

// Residual add, RMSNorm and the per-token quantiser in one pass over a row (the quantiser fused into the operator in
// front of it, Sec. 6.1; the norm is LLaMA's):
//   r = fp16(fp32(res) + fp32(x))  (r = x without a residual),  y = fp16(fp32(r) * rsqrt(mean r^2 + eps) * fp32(g)),
//   (xq, s_a) = the per-token quantiser of quantize_act_kernel applied to y.
// The mean of squares is an fp32 sum (per thread, then over the workgroup), the reciprocal square root the hardware's
// square root (within one ulp) and a correctly rounded division.  r and y are written where the caller wants them (the residual stream goes on; y
// is for inspection), otherwise the only traffic is x, res, g in and the codes out.  A thread keeps its chunks of the
// row in registers (K <= 16384); longer rows take what is beyond from r as written, or from the inputs again, with the
// same bits.
// One reduction, of the squares and of |r g| together, where the scale needs no y (absmax_of_norm), the gain requested behind the
// chunk it belongs to; a thread has as many chunks as the row's length asks for.  Bound by latency below some 300 rows, by the vector
// ALU and memory beyond.  With two reductions, conversions around every product and always 1024 x 2 or 256 x 8 chunks, and now,
// residual added, back to back: 200 x 4096 4.7 -> 3.6 us, 333 x 4096 5.6 -> 4.5, 1024 x 5120 11.2 -> 9.9 (3.7 TB/s), 2048 x 8192 30.6 -> 27.0.
// Few rows: the order of the sum is that of 1024 threads, but up to K = 8192 on 512 of them, chain q of a thread being the thread
// 512 q further on; half the waves, and none with nothing to do.  On 1024 threads one reduction was slower than two, without a residual
// above all (16 x 8192 3.8 us with two, 4.1 with one, 3.6 so; 1 x 8192 3.5, 3.85, 3.3; with the residual 16 x 5120 3.8, 3.8, 3.5).
// From two to six chunks a thread x, residual and gains of all of them are asked for ahead of the first sum, as buffer loads with no branch
// between (with a branch around each chunk the gain of a chunk was asked for behind its x, the next chunk behind both): 16 x 5120 3.43 ->
// 3.14 us, 333 x 4096 4.65 -> 4.53, 1024 x 5120 10.15 -> 9.67, 2048 x 8192 25.5 -> 23.8.  With one chunk there is nothing to gather, the
// waves past a short row's end load nothing, and the margin of the row maximum is the shorter chain: 1 x 2048 2.33 us where loads without
// branches and a margin per value take 2.50, 64 x 2048 2.66 and 2.82, 128 x 1024 2.67 and 2.85; 64 x 4096 level.
template <int THREADS, int CACHE, int CHAINS = 1>
__global__ __launch_bounds__(THREADS) void add_rmsnorm_quantize_kernel(const uint16_t *x, const uint16_t *res,
                                                                     const uint16_t *__restrict__ gamma, float eps,
                                                                     uint16_t *r_out, uint16_t *__restrict__ y_out,
                                                                     int8_t *__restrict__ xq, float *__restrict__ s_a, int K) {
    constexpr int kWaves = THREADS / 64;
    __shared__ float scratch[kWaves];
    __shared__ float scratch_sum[CHAINS * kWaves];
    __shared__ float scratch_top[kWaves];
    const int m = blockIdx.x;
    const int chunks = K >> 3;
    const v4u *xs = (const v4u *)(x + (size_t)m * K);
    const v4u *rs = res ? (const v4u *)(res + (size_t)m * K) : nullptr;
    const v4u *gs = (const v4u *)gamma;
    auto r_chunk = [&](int c) { return rs ? add_halves8(rs[c], xs[c]) : xs[c]; };
    // what the later passes take for a chunk beyond the registers: r as written (r_out may be x or res themselves, which
    // this thread has then overwritten), else the same sum again
    auto r_again = [&](int c) { return r_out ? ((const v4u *)(r_out + (size_t)m * K))[c] : r_chunk(c); };

    constexpr bool kKeepGains = CACHE <= 6;  // longer rows fetch them again
    // Waves past the row's end skip the arithmetic, which leaves its issue slots to the others, where the rows are few (16 x 12288
    // 4.5 -> 4.3 us); with many rows the branches cost 20 % at K = 9216.
    constexpr bool kSkip = CHAINS > 1 || THREADS == 1024;
    v4u cache[CACHE], gain[kKeepGains ? CACHE : 1];
    float ss[CHAINS] = {};
    unsigned top = 0u;
    if constexpr (kKeepGains && CACHE > 1) {
        const __amdgpu_buffer_rsrc_t x_row = row_buffer(xs, chunks), res_row = row_buffer(rs, rs ? chunks : 0), g_row = row_buffer(gs, chunks);
        v4u res_chunk[CACHE];
#pragma unroll
        for (int i = 0; i < CACHE; ++i) {
            const int c = threadIdx.x + i * THREADS;
            cache[i] = row_chunk(x_row, c);
            res_chunk[i] = row_chunk(res_row, c);
        }
#pragma unroll
        for (int i = 0; i < CACHE; ++i) gain[kKeepGains ? i : 0] = row_chunk(g_row, threadIdx.x + i * THREADS);
        __builtin_amdgcn_sched_barrier(0);
        if (rs) {  // r = x as it is otherwise, -0 too
#pragma unroll
            for (int i = 0; i < CACHE; ++i) cache[i] = add_halves8(res_chunk[i], cache[i]);
        }
#pragma unroll
        for (int i = 0; i < CACHE; ++i) {
            const int c = threadIdx.x + i * THREADS;
            if (r_out && c < chunks) ((v4u *)(r_out + (size_t)m * K))[c] = cache[i];
            if (kSkip && c >= chunks) continue;
            ss[i % CHAINS] = add_squares8(cache[i], ss[i % CHAINS]);
            top = absmax_products8(cache[i], gain[kKeepGains ? i : 0], top);
        }
    } else {
#pragma unroll
        for (int i = 0; i < CACHE; ++i) {
            const int c = threadIdx.x + i * THREADS;
            cache[i] = v4u{0, 0, 0, 0};
            v4u gn = v4u{0, 0, 0, 0};
            if (c < chunks) {
                cache[i] = r_chunk(c);
                gn = gs[c];
                if (r_out) ((v4u *)(r_out + (size_t)m * K))[c] = cache[i];
            }
            if (kSkip && c >= chunks) continue;
            ss[i % CHAINS] = add_squares8(cache[i], ss[i % CHAINS]);
            top = absmax_products8(cache[i], gn, top);
            if (kKeepGains) gain[kKeepGains ? i : 0] = gn;
        }
    }
    for (int c0 = threadIdx.x + CACHE * THREADS; c0 < chunks; c0 += CHAINS * THREADS)
#pragma unroll
        for (int q = 0; q < CHAINS; ++q) {
            const int c = c0 + q * THREADS;
            if (c < chunks) {
                const v4u r = r_chunk(c);
                if (r_out) ((v4u *)(r_out + (size_t)m * K))[c] = r;
                ss[q] = add_squares8(r, ss[q]);
                top = absmax_products8(r, gs[c], top);
            }
        }
    // over the workgroup: DPP steps inside the wave, the waves' sums in wave order, chain by chain
#pragma unroll
    for (int q = 0; q < CHAINS; ++q) ss[q] = wave_sum(ss[q]);
    const float wave_top = wave_max_nonneg(__uint_as_float(top));
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int q = 0; q < CHAINS; ++q) scratch_sum[q * kWaves + (threadIdx.x >> 6)] = ss[q];
        scratch_top[threadIdx.x >> 6] = wave_top;
    }
    __syncthreads();
    float total = 0.f;
    unsigned row_top = 0u;
#pragma unroll
    for (int w = 0; w < CHAINS * kWaves; ++w) total += scratch_sum[w];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) row_top = max(row_top, __float_as_uint(scratch_top[w]));
    const float inv = rms_inverse(total, K, eps);
    auto y_chunk = [&](int c, v4u r) { return norm_scale8(r, inv, gs[c]); };
#pragma unroll
    for (int i = 0; i < CACHE; ++i) {  // from here on the cache holds y
        const int c = threadIdx.x + i * THREADS;
        if (kSkip && c >= chunks) continue;
        if (kKeepGains)
            cache[i] = norm_scale8(cache[i], inv, gain[kKeepGains ? i : 0]);
        else if (c < chunks)
            cache[i] = y_chunk(c, cache[i]);
    }
    float amax;
    if (!absmax_of_norm(__uint_as_float(row_top), inv, &amax)) {  // the same for all threads
        unsigned amax2 = 0u;
#pragma unroll
        for (int i = 0; i < CACHE; ++i)
            if ((int)threadIdx.x + i * THREADS < chunks) amax2 = absmax8_packed(cache[i], amax2);
        for (int c = threadIdx.x + CACHE * THREADS; c < chunks; c += THREADS) amax2 = absmax8_packed(y_chunk(c, r_again(c)), amax2);
        amax = block_max<THREADS, true>(absmax_packed_value(amax2), scratch);
    }

    const RowQuantizer rq(amax, 127.0f, -127.f, 127.f);
    if (threadIdx.x == 0) s_a[m] = rq.scale;
    const bool zero_row = amax == 0.f;
    v2u *dst = (v2u *)(xq + (size_t)m * K);
    auto emit = [&](int c, v4u y) {
        if (y_out) ((v4u *)(y_out + (size_t)m * K))[c] = y;
        v2u o = v2u{0, 0};
        if (!zero_row) {
            float yf[8];
            halves8(y, yf);
            o = rq.packed8_own_max<(CACHE > 1)>(yf);
        }
        dst[c] = o;
    };
#pragma unroll
    for (int i = 0; i < CACHE; ++i) {
        const int c = threadIdx.x + i * THREADS;
        if (c < chunks) emit(c, cache[i]);
    }
    for (int c = threadIdx.x + CACHE * THREADS; c < chunks; c += THREADS) emit(c, y_chunk(c, r_again(c)));
}

template <int THREADS, int CACHE, int CHAINS = 1>
static void launch_norm(const void *x, const void *res, const void *gamma, float eps, void *r_out, void *y_out, int8_t *xq, float *s_a,
                        int M, int K, hipStream_t stream) {
    hipLaunchKernelGGL((add_rmsnorm_quantize_kernel<THREADS, CACHE, CHAINS>), dim3(M), dim3(THREADS), 0, stream, (const uint16_t *)x,
                       (const uint16_t *)res, (const uint16_t *)gamma, eps, (uint16_t *)r_out, (uint16_t *)y_out, xq, s_a, K);
}

hipError_t launch_add_rmsnorm_quantize(const void *x, const void *res, const void *gamma, float eps, void *r_out, void *y_out,
                                       int8_t *xq, float *s_a, int M, int K, hipStream_t stream) {
    const int chunks = K >> 3;
#define W4A8_NORM(...) launch_norm<__VA_ARGS__>(x, res, gamma, eps, r_out, y_out, xq, s_a, M, K, stream)
    if (M <= kFewRows) {
        if (chunks <= 512) W4A8_NORM(512, 1);
        else if (chunks <= 1024) W4A8_NORM(512, 2, 2);
        else W4A8_NORM(1024, 2);
    } else if (M <= kSomeRows) {
        if (chunks <= 512) W4A8_NORM(512, 1);
        else if (chunks <= 1024) W4A8_NORM(512, 2);
        else W4A8_NORM(512, 4);
    } else {
        switch ((chunks + 255) / 256) {
            case 1: W4A8_NORM(256, 1); break;
            case 2: W4A8_NORM(256, 2); break;
            case 3: W4A8_NORM(256, 3); break;
            case 4: W4A8_NORM(256, 4); break;
            case 5: W4A8_NORM(256, 5); break;
            case 6: W4A8_NORM(256, 6); break;
            default: W4A8_NORM(256, 8);
        }
    }
#undef W4A8_NORM
    return hipGetLastError();
}

hipError_t launch_quantize_act(const void *x, long long ldx, int8_t *xq, float *s_a, int M, int K, hipStream_t stream) {
    // up to half a row per compute unit the rows are spread over four times the threads
    if (M <= kFewRows)
        hipLaunchKernelGGL((quantize_act_kernel<1024, 2>), dim3(M), dim3(1024), 0, stream, (const uint16_t *)x, xq, s_a, K, ldx);
    else if (M <= kSomeRows)
        hipLaunchKernelGGL((quantize_act_kernel<512, 4>), dim3(M), dim3(512), 0, stream, (const uint16_t *)x, xq, s_a, K, ldx);
    else
        hipLaunchKernelGGL((quantize_act_kernel<kRowThreads, kCache>), dim3(M), dim3(kRowThreads), 0, stream, (const uint16_t *)x,
                           xq, s_a, K, ldx);
    return hipGetLastError();
}

hipError_t launch_quantize_weights(const void *w, uint8_t *wp, float *s_w, int N, int K, hipStream_t stream) {
    if (K <= kShortRow)
        hipLaunchKernelGGL((quantize_weights_kernel<128, kShortRow / (128 * 8)>), dim3(N), dim3(128), 0, stream, (const uint16_t *)w, wp,
                           s_w, K);
    else
        hipLaunchKernelGGL((quantize_weights_kernel<kRowThreads, kCache>), dim3(N), dim3(kRowThreads), 0, stream,
                           (const uint16_t *)w, wp, s_w, K);
    return hipGetLastError();
}

hipError_t launch_quantize_weights_clip(const void *w, const float *gamma, const float *beta, uint8_t *wp, float *s_w, int N,
                                        int K, hipStream_t stream) {
    hipLaunchKernelGGL(quantize_weights_clip_kernel, dim3(N), dim3(kRowThreads), 0, stream, (const uint16_t *)w, gamma, beta,
                       wp, s_w, K);
    return hipGetLastError();
}

hipError_t launch_silu_mul(const void *gate_up, void *h, int M, int I, hipStream_t stream) {
    const int chunks = I >> 3;
    dim3 grid((chunks + kRowThreads - 1) / kRowThreads, M);
    hipLaunchKernelGGL(silu_mul_kernel, grid, dim3(kRowThreads), 0, stream, (const uint16_t *)gate_up, (uint16_t *)h, I);
    return hipGetLastError();
}

hipError_t launch_silu_mul_quantize(const void *gate_up, int8_t *xq, float *s_a, int M, int I, hipStream_t stream) {
    hipLaunchKernelGGL(silu_mul_quantize_kernel, dim3(M), dim3(kFusedThreads), 0, stream, (const uint16_t *)gate_up, xq, s_a, I);
    return hipGetLastError();
}

}  // namespace w4a8
